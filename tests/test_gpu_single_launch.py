"""The single-launch form (own-segment tiles and prefix walk in one kernel) and the walk without a
stop rule, at the places where their tile pipeline changes over: odd and even numbers of
own-segment tiles, wavefronts that need fewer of them than their workgroup, workgroups without
rows, budgets of one tile, an odd and an even last tile, and logits that move the softmax
reference in the middle of a walk."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

from oracle import s2o_oracle as orc
from paper_2602_22575_amd import inputs
import gpu_util as gu
import parity


def _inputs(L, S, BM, scale_up=0):
    w = inputs.workload("llama8k", L=L, S=S, H=2, Hkv=1, BM=BM, seed=L + S)
    Qb, Kb, Vb = inputs.make_qkv(w)
    # queries times 2**scale_up, exactly: one more in the exponent field of a normal number
    Qb = np.where(Qb & 0x7f80 != 0, Qb + np.uint16(scale_up << 7), Qb).astype(np.uint16)
    return w, (Qb, Kb, Vb), tuple(gu.to_dev(x) for x in (Qb, Kb, Vb))


@pytest.mark.parametrize("L,S,BM", [(192, 64, 64), (576, 192, 64), (640, 128, 128), (1152, 384, 128), (960, 320, 64)])
@pytest.mark.parametrize("use_q_perm", [0, 1])
def test_own_segment_then_prefix(gpu, L, S, BM, use_q_perm):
    w, (Qb, Kb, Vb), (Qd, Kd, Vd) = _inputs(L, S, BM)
    plan, pg = gu.gpu_plan(w, Qd, Kd)
    for stop_mode, tau, budget in ((0, 0.0, 0), (0, 0.05, 0), (1, 0.05, 0), (2, 0.0, 0), (2, 0.0, 1), (0, 0.02, 2)):
        print(f"case: single launch L={L} S={S} BM={BM} q_perm={use_q_perm} stop_mode={stop_mode} tau={tau} "
              f"budget={budget}", flush=True)
        Ob, c, s = gu.gpu_attention(w, Qd, Kd, Vd, plan.q_perm, plan.kv_perm, tau, stop_mode, use_q_perm=use_q_perm,
                                    two_pass=False, max_tiles=budget)
        parity.check_attention(w, Qb, Kb, Vb, pg["q_perm"] if use_q_perm else None, pg["kv_perm"], tau, stop_mode, Ob,
                               c, s, use_q_perm=bool(use_q_perm), max_tiles=budget)


@pytest.mark.parametrize("two_pass", [True, False])
def test_no_stop_rule_with_rising_logits(gpu, two_pass):
    """Rows of KV_perm turned round (the largest scores last) and logits of a standard deviation of
    about 16: the reference has to follow the running maximum through the walk."""
    w, (Qb, Kb, Vb), (Qd, Kd, Vd) = _inputs(1280, 256, 64, scale_up=4)
    plan, pg = gu.gpu_plan(w, Qd, Kd)
    kv = pg["kv_perm"].copy()
    for n in range(1, w.N):
        o = orc.kv_row_offset(n, w.S)
        kv[:, :, o:o + n * w.S] = kv[:, :, o:o + n * w.S][:, :, ::-1]
    kvd = plan.kv_perm.new_tensor(kv)
    Ob, c, s = gu.gpu_attention(w, Qd, Kd, Vd, plan.q_perm, kvd, 0.0, 2, two_pass=two_pass)
    parity.check_attention(w, Qb, Kb, Vb, pg["q_perm"], kv, 0.0, 2, Ob, c, s)
    assert np.all(s == 0)


@pytest.mark.parametrize("L", [64, 128, 192, 448])
def test_contiguous_attention_over_few_tiles(gpu, L):
    w, (Qb, Kb, Vb), (Qd, Kd, Vd) = _inputs(L, L, 64)
    Ob, c, s = gu.gpu_attention(w, Qd, Kd, Vd, None, None, 0.0, 2, use_q_perm=0, non_causal=1)
    Q, K, V = (parity.to_f64(x) for x in (Qb, Kb, Vb))
    for h in range(w.H):
        x = Q[0, h] @ K[0, h // w.G].T / np.sqrt(w.D)
        p = np.exp(x - x.max(axis=1, keepdims=True))
        ref = (p / p.sum(axis=1, keepdims=True)) @ V[0, h // w.G]
        assert np.abs(parity.to_f64(Ob)[0, h] - ref).max() <= parity.O_MAX_ABS
    assert np.all(c == L // 64) and np.all(s == 0)
