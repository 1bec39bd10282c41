"""The matrix products of the attention kernels are assembly texts, around which the compiler places no wait states of
its own: no vector instruction may write an operand of one in the two slots in front of it, and before a result is in its
registers nothing may touch it but a product that adds to exactly that accumulator: not a product that takes it as a
factor, nor one whose accumulator overlaps it in part.  The instructions that the compiler put there are checked."""
import os
import re
import subprocess

import pytest

from paper_2602_22575_amd import build as b
from test_asm_reads_in_flight import _registers, kernels

# A slot is 4 clocks.  v_mfma_f32_16x16x32_bf16 takes 4 passes of 4 clocks: the product behind it cannot start earlier than
# 4 slots after it.  Around products of its own the compiler leaves 8 slots before anything reads the result (another
# product's factor included) and 2 between a vector instruction and the product that reads what it wrote
# (test_the_slots_are_the_compilers); 3 more are kept behind a product here.
RESULT_SLOTS, PRODUCT_SLOTS, OPERAND_SLOTS = 8 + 3, 4, 2


def _next(body, label, i):
    op, _, args = body[i].partition(" ")
    if op == "s_endpgm":
        return []
    if op == "s_branch":
        return [label[args.strip()]]
    return [i + 1] + ([label[args.strip()]] if op.startswith("s_cbranch") else [])


def _operands(args):
    """Register sets of a product: result, factors, accumulator that it adds to."""
    d, a, b, c = (_registers(x) for x in args.split(",")[:4])
    return d, a | b, c


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
        # `at`: slots behind `start` at which an instruction is issued at the earliest, `last`: the latest product's
        todo, seen = [(i, 1, 0 if product else -PRODUCT_SLOTS) for i in _next(body, label, start)], set()
        while todo:
            i, at, last = todo.pop()
            if (i, at, last) in seen or at > (RESULT_SLOTS if product else OPERAND_SLOTS):
                continue
            seen.add((i, at, last))
            if body[i].endswith(":"):
                todo.append((i + 1, at, last))
                continue
            o, _, a = body[i].partition(" ")
            if o.startswith("v_mfma"):
                d, factors, c = _operands(a)
                at = last = max(at, last + PRODUCT_SLOTS)
                if at > (RESULT_SLOTS if product else OPERAND_SLOTS):
                    pass
                elif product:
                    if result & factors or any(result & x and result != x for x in (c, d)):
                        bad.add((line, body[i]))
                elif result & (factors | c):
                    bad.add((line, body[i]))
            elif product and not o.startswith("s_") and result & _registers(a):
                bad.add((line, body[i]))
            todo += [(n, at + (int(a) + 1 if o == "s_nop" else 1), last) for n in _next(body, label, i)]
    return sorted(bad)


def _assembly(source, out):
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    subprocess.run([hipcc, *b.FLAGS, "--cuda-device-only", "-S", str(source), "-o", str(out)], check=True, capture_output=True)
    return kernels(out.read_text())


@pytest.mark.parametrize("source", ["prefix.hip", "local.hip"])
def test_products_keep_their_distance(source, tmp_path):
    found = _assembly(os.path.join(b.CSRC, source), tmp_path / (source + ".s"))
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
    ([PRODUCT, PRODUCT], 0),                                                     # the same accumulator
    ([PRODUCT, "v_mfma_f32_16x16x32_bf16 v[4:7], v[0:3], v[12:15], v[4:7]"], 1),      # a result as a factor
    ([PRODUCT, "v_mfma_f32_16x16x32_bf16 v[4:7], v[8:11], v[0:3], 0"], 1),
    ([PRODUCT, "v_mfma_f32_16x16x32_bf16 v[2:5], v[8:11], v[12:15], v[2:5]"], 1),     # accumulators that overlap in part
    ([PRODUCT, "v_mfma_f32_16x16x32_bf16 v[2:5], v[8:11], v[12:15], 0"], 1),
    ([PRODUCT, "s_nop 10", "v_mfma_f32_16x16x32_bf16 v[4:7], v[0:3], v[12:15], v[4:7]"], 0),
    # a product holds the next one up from its own start on: not for the slots that others have filled
    ([PRODUCT, "s_nop 2", PRODUCT.replace("v[0:3]", "v[4:7]"), "s_nop 4", "v_mov_b32_e32 v9, v0"], 1),
    ([PRODUCT, "s_nop 2", PRODUCT.replace("v[0:3]", "v[4:7]"), "s_nop 6", "v_mov_b32_e32 v9, v0"], 0),
])
def test_the_check_sees_what_it_looks_for(body, bad):
    assert len(too_close(body + ["s_endpgm"])) == bad


ONE_PRODUCT = """#include <hip/hip_runtime.h>
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
__device__ f32x4 product(bf16x8 a, bf16x8 b) { return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, f32x4{}, 0, 0, 0); }
extern "C" __global__ void stored(const bf16x8* a, f32x4* o) { o[0] = product(a[0], a[1]); }
extern "C" __global__ void factor(const bf16x8* a, f32x4* o) { o[0] = product(__builtin_bit_cast(bf16x8, product(a[0], a[1])), a[1]); }
extern "C" __global__ void written(const bf16x8* a, f32x4* o) {
  f32x4 x = __builtin_bit_cast(f32x4, a[0]);
  for (int i = 0; i < 4; ++i) asm volatile("" : "+v"(x[i]));
  for (int i = 0; i < 4; ++i) x[i] *= 3.f;
  o[0] = product(__builtin_bit_cast(bf16x8, x), a[1]);
}
"""


def test_the_slots_are_the_compilers(tmp_path):
    source = tmp_path / "one.hip"
    source.write_text(ONE_PRODUCT)
    found = _assembly(source, tmp_path / "one.s")

    def idle(body, at):                                    # the slots of an s_nop at that place
        assert body[at].startswith("s_nop"), body
        return int(body[at].split()[1]) + 1

    for name in ("stored", "factor"):
        first = next(i for i, line in enumerate(found[name]) if line.startswith("v_mfma"))
        assert idle(found[name], first + 1) == 8 <= RESULT_SLOTS, found[name]
    first = next(i for i, line in enumerate(found["written"]) if line.startswith("v_mfma"))
    assert idle(found["written"], first - 1) <= OPERAND_SLOTS, found["written"]
