"""LDS reads that the attention kernels issue in assembly texts are in flight while the compiler takes their
registers as loaded: between such a read and the wait that covers it nothing may touch them, not even a copy or a
spill.  Nothing in the source can ask the compiler for that, so the instructions it made are checked, along
every path of every kernel."""
import os
import re
import subprocess

import pytest

from paper_2602_22575_amd import build as b

REGISTERS = re.compile(r"\b([va])(?:(\d+)\b|\[(\d+):(\d+)\])")
HAS_RESULT = re.compile(r"ds_(read|bpermute|permute|swizzle|\w+_rtn)")


def _registers(text):
    out = set()
    for kind, one, lo, hi in REGISTERS.findall(text):
        out.update((kind, i) for i in range(int(lo or one), int(hi or one) + 1))
    return out


def kernels(assembly):
    """{name: [instruction or label, ...]} of a device assembly listing."""
    out, body = {}, None
    for line in assembly.splitlines():
        line = line.split(";")[0].strip()
        m = re.fullmatch(r"(\w+):", line)
        if m and not line.startswith(".L"):
            body = out.setdefault(m[1], [])
        elif body is not None and (line.startswith(".LBB") or (line and not line.startswith("."))):
            body.append(line)
    return {k: v for k, v in out.items() if any(i.startswith("s_endpgm") for i in v)}


def touched_in_flight(body):
    """Instructions that name a register which an LDS read in flight has yet to write: [(index, instruction)].
    LDS instructions complete in order; lgkmcnt(n) leaves at most n of them."""
    label = {line[:-1]: i for i, line in enumerate(body) if line.startswith(".LBB")}
    bad, seen, todo = set(), set(), [(0, ())]
    while todo:
        i, flight = todo.pop()
        while i < len(body):
            line = body[i]
            if line.endswith(":"):
                if (i, flight) in seen:
                    break
                seen.add((i, flight))
                i += 1
                continue
            op, _, args = line.partition(" ")
            if op == "s_waitcnt":
                m = re.search(r"lgkmcnt\((\d+)\)", args)
                if m:
                    flight = flight[max(0, len(flight) - int(m[1])):]
            elif op == "s_endpgm":
                break
            elif op in ("s_branch",) or op.startswith("s_cbranch"):
                target = label[args.strip()]
                if op == "s_branch":
                    i = target
                    continue
                todo.append((target, flight))
            else:
                assert op not in ("s_setpc_b64", "s_swappc_b64") and not op.startswith("flat_"), line
                used = _registers(args)
                if used & set().union(*flight):
                    bad.add((i, line))
                if op.startswith("ds_"):
                    flight += (frozenset(_registers(args.split(",")[0])) if HAS_RESULT.match(op) else frozenset(),)
            i += 1
    return sorted(bad)


@pytest.mark.parametrize("source", ["prefix.hip", "local.hip"])
def test_nothing_touches_a_read_in_flight(source, tmp_path):
    out = tmp_path / (source + ".s")
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    subprocess.run([hipcc, *b.FLAGS, "--cuda-device-only", "-S", os.path.join(b.CSRC, source), "-o", str(out)],
                   check=True, capture_output=True)
    found = kernels(out.read_text())
    assert len(found) == {"prefix.hip": 8, "local.hip": 1}[source]
    for name, body in found.items():
        assert sum(i.startswith("ds_read") for i in body) > 50, name
        assert not touched_in_flight(body), (name, touched_in_flight(body)[:5])


READ = ["ds_read_b128 v[0:3], v8", "ds_read_b128 v[4:7], v8 offset:512"]


@pytest.mark.parametrize("body,bad", [
    (READ + ["s_waitcnt lgkmcnt(1)", "v_mov_b32_e32 v9, v3", "s_waitcnt lgkmcnt(0)", "v_mov_b32_e32 v9, v7"], 0),
    (READ + ["s_waitcnt lgkmcnt(1)", "v_mov_b32_e32 v9, v4"], 1),                        # a copy
    (READ + ["scratch_store_dwordx4 off, v[0:3], off", "s_waitcnt vmcnt(0)"], 1),        # a spill
    (READ + ["v_mov_b32_e32 v2, 0"], 1),                                                 # written too early
    (READ + ["ds_write_b32 v10, v11", "s_waitcnt lgkmcnt(2)", "v_mov_b32_e32 v9, v0", "v_mov_b32_e32 v9, v4"], 1),
    (["s_cbranch_scc0 .LBB0_2", *READ, ".LBB0_2:", "v_mov_b32_e32 v9, v0"], 1),          # on one of two paths
    ([".LBB0_1:", "v_accvgpr_write_b32 a0, v4", *READ, "s_waitcnt lgkmcnt(1)", "s_cbranch_scc1 .LBB0_1"], 2),   # around a loop
])
def test_the_check_sees_what_it_looks_for(body, bad):
    assert len(touched_in_flight(body + ["s_endpgm"])) == bad
