"""Assembly texts in the kernels keep their own wait states: the compiler's hazard recogniser does
not look into a text, nor does it count on one."""
import glob
import os
import re

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2602_22575_amd", "csrc")
SOURCES = sorted(glob.glob(os.path.join(CSRC, "*.h*")))
TAKES_A_MASK = re.compile(r"v_(addc|subb|subbrev|cndmask)")


def asm_texts(source):
    """Instructions of every asm statement that has some: [(line number, [instruction, ...])]."""
    texts = []
    for m in re.finditer(r"\basm\b(?:\s+volatile)?\s*\(((?:\s*\"(?:[^\"\\]|\\.)*\")+)", source):
        text = "".join(re.findall(r"\"((?:[^\"\\]|\\.)*)\"", m.group(1)))
        ins = [i.strip() for i in text.replace("\\n", "\n").replace("\\t", "\t").split("\n") if i.strip()]
        if ins:
            texts.append((source.count("\n", 0, m.start()) + 1, ins))
    return texts


@pytest.mark.parametrize("path", SOURCES, ids=os.path.basename)
def test_masks_are_read_behind_their_wait_states(path):
    """A vector instruction may read a mask register no earlier than two wait states after the
    comparison (or lane read) that wrote it, and a data-parallel move a vector register two after it
    was written: a text with an add-with-carry or select starts and ends with `s_nop 1` at least."""
    with open(path) as f:
        texts = asm_texts(f.read())
    for line, ins in texts:
        if any(TAKES_A_MASK.match(i) for i in ins):
            for end in (ins[0], ins[-1]):
                m = re.fullmatch(r"s_nop (\d+)", end)
                assert m and int(m.group(1)) >= 1, f"{os.path.basename(path)}:{line}: {ins}"


def test_the_scan_sees_the_texts():
    texts = [ins for path in SOURCES for _, ins in asm_texts(open(path).read())]
    assert sum(len(t) for t in texts) > 20 and any(TAKES_A_MASK.match(i) for t in texts for i in t)
