"""The matrix products of the attention kernels are assembly texts, around which the compiler places no wait states of
its own: no vector instruction may write an operand of one in the two slots in front of it, and nothing but another
product may touch a result before it is in its registers.  The instructions that the compiler put there are checked."""
import os
import re
import subprocess

import pytest

from paper_2602_22575_amd import build as b
from test_asm_reads_in_flight import _registers, kernels

# v_mfma_f32_16x16x32_bf16 takes 8 passes: 11 slots before a vector or memory instruction reads or overwrites its result.  A product
# that follows holds its successor up for four passes at least.
RESULT_SLOTS, PRODUCT_SLOTS, OPERAND_SLOTS = 11, 4, 2


def _slots(line):
    op, _, args = line.partition(" ")
    return int(args) + 1 if op == "s_nop" else PRODUCT_SLOTS if op.startswith("v_mfma") else 1


def _next(body, label, i):
    op, _, args = body[i].partition(" ")
    if op == "s_endpgm":
        return []
    if op == "s_branch":
        return [label[args.strip()]]
    return [i + 1] + ([label[args.strip()]] if op.startswith("s_cbranch") else [])


def too_close(body):
    """[(instruction, the one too close behind it)], along every path."""
    label = {line[:-1]: i for i, line in enumerate(body) if line.endswith(":")}
    bad = set()
    for start, line in enumerate(body):
        op, _, args = line.partition(" ")
        if not op.startswith("v_") or op.startswith(("v_cmp", "v_readfirstlane", "v_readlane")):
            continue
        product = op.startswith("v_mfma")
        swap = "swap" in op                                # writes both of its operands
        result = _registers(args if swap else args.split(",")[0])
        todo, seen = [(i, 0) for i in _next(body, label, start)], set()
        while todo:
            i, slots = todo.pop()
            if (i, slots) in seen or slots >= (RESULT_SLOTS if product else OPERAND_SLOTS):
                continue
            seen.add((i, slots))
            if body[i].endswith(":"):
                todo.append((i + 1, slots))
                continue
            o, _, a = body[i].partition(" ")
            if product and not o.startswith(("v_mfma", "s_")) and result & _registers(a):
                bad.add((line, body[i]))
            if not product and o.startswith("v_mfma") and result & _registers(a.split(",", 1)[1]):
                bad.add((line, body[i]))
            todo += [(n, slots + _slots(body[i])) for n in _next(body, label, i)]
    return sorted(bad)


@pytest.mark.parametrize("source", ["prefix.hip", "local.hip"])
def test_products_keep_their_distance(source, tmp_path):
    out = tmp_path / (source + ".s")
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    subprocess.run([hipcc, *b.FLAGS, "--cuda-device-only", "-S", os.path.join(b.CSRC, source), "-o", str(out)],
                   check=True, capture_output=True)
    found = kernels(out.read_text())
    assert found
    for name, body in found.items():
        products = {i.partition(" ")[0] for i in body if i.startswith("v_mfma")}
        assert products == {"v_mfma_f32_16x16x32_bf16"}, (name, products)
        assert not too_close(body), (name, too_close(body)[:5])


PRODUCT = "v_mfma_f32_16x16x32_bf16 v[0:3], v[8:11], v[12:15], v[0:3]"


@pytest.mark.parametrize("body,bad", [
    (["v_mov_b32_e32 v9, v20", "s_waitcnt lgkmcnt(0)", PRODUCT], 1),
    (["v_mov_b32_e32 v9, v20", "s_waitcnt lgkmcnt(0)", "s_nop 0", PRODUCT], 0),
    (["v_mov_b32_e32 v2, v20", PRODUCT], 1),                                     # the accumulator as well
    (["v_permlane32_swap_b32_e32 v20, v9", PRODUCT], 1),
    ([PRODUCT, "s_nop 9", "v_mul_f32 v3, v4, v3"], 1),
    ([PRODUCT, "s_nop 10", "v_mul_f32 v3, v4, v3"], 0),
    ([PRODUCT, PRODUCT.replace("v[0:3]", "v[4:7]"), "s_nop 6", "global_store_dword v20, v3, s[0:1]"], 0),
    ([PRODUCT, "s_cbranch_scc0 .LBB0_2", "s_nop 15", ".LBB0_2:", "v_mov_b32_e32 v9, v0"], 1),
])
def test_the_check_sees_what_it_looks_for(body, bad):
    assert len(too_close(body + ["s_endpgm"])) == bad
