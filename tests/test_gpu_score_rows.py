"""Scores and key order where a KV head has several groups of 128 rows: full and partly filled groups and row
blocks, heads per KV head that divide a block of 32 rows and that do not, one group more and one less;
rows by segment (up to 255 of them, with causality) and by head."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

from paper_2602_22575_amd import inputs
import gpu_util as gu
import parity


@pytest.mark.parametrize("H,Hkv,N", [(4, 1, 32), (4, 1, 33), (3, 1, 50), (6, 2, 64), (1, 1, 129), (10, 2, 77), (3, 1, 255), (3, 1, 256)])
@pytest.mark.parametrize("non_causal", [0, 1])
def test_scores_of_several_row_groups(gpu, H, Hkv, N, non_causal):
    S, L = 64, 64 * N
    w = inputs.workload("llama8k", L=L, S=S, H=H, Hkv=Hkv, seed=L + H)
    Qb, Kb, _ = inputs.make_qkv(w)
    print(f"case: H={H} Hkv={Hkv} N={N} non_causal={non_causal}", flush=True)
    _, pg = gu.gpu_plan(w, gu.to_dev(Qb), gu.to_dev(Kb), non_causal=non_causal)
    K = parity.to_f64(Kb)
    for h in range(H):
        k = K[0, h // w.G]
        for n in range(0 if non_causal else 1, N):
            m = L if non_causal else n * S
            o = n * L if non_causal else S * n * (n - 1) // 2
            s = pg["s_k"][0, h, o:o + m]
            q = pg["q_mean"][0, h, n].astype(np.float64)
            # the protocol's bound: fp32 sums of 128 exact products
            assert np.all(np.abs(s - k[:m] @ q) <= 1e-6 * (np.abs(k[:m]) @ np.abs(q)) + 1e-6), (h, n)
            assert np.array_equal(pg["kv_perm"][0, h, o:o + m], np.argsort(-s, kind="stable")), (h, n)
