"""Rows that fit one sort: the edges of the sort's shapes (2048, 4096, 6656, 7168, 10240 and 13312 keys), with at most one
row a CU and with more, where a workgroup takes a second and third row, the last ones of them short.  The maps
must equal the stable argsort of the plan's own scores entry for entry."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

from paper_2602_22575_amd import inputs
import gpu_util as gu


@pytest.mark.parametrize("H", [1, 9])
@pytest.mark.parametrize("L,S,non_causal", [
    (2112, 64, 0), (2176, 64, 0), (4160, 64, 0), (4224, 64, 0), (6720, 64, 0), (6784, 64, 0), (7232, 64, 0), (7296, 64, 0),
    (10304, 64, 0), (10368, 64, 0), (13376, 64, 0), (4096, 128, 1), (7168, 128, 1), (10240, 256, 1), (13312, 256, 1)])
def test_every_row(gpu, L, S, non_causal, H):
    w = inputs.workload("llama8k", L=L, S=S, H=H, Hkv=1, seed=L + H)
    Qb, Kb, _ = inputs.make_qkv(w)
    print(f"case: whole rows L={L} S={S} H={H} non_causal={non_causal}", flush=True)
    _, pg = gu.gpu_plan(w, gu.to_dev(Qb), gu.to_dev(Kb), non_causal=non_causal)
    for h in range(H):
        for n in range(0 if non_causal else 1, w.N):
            at, ln = (n * L, L) if non_causal else (S * n * (n - 1) // 2, n * S)
            sk = pg["s_k"][0, h, at:at + ln]
            assert np.array_equal(pg["kv_perm"][0, h, at:at + ln], np.argsort(-sk, kind="stable")), (h, n)
