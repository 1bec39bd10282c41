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


def _bf16(x):
    """Nearest bf16 (ties to even) of finite float64 values, as bits."""
    u = np.asarray(x, np.float32).view(np.uint32)
    return ((u + 0x7fff + ((u >> 16) & 1)) >> 16).astype(np.uint16)


def _online(tiles, V, lazy):
    """Online softmax over (logits base 2, rows of V) tiles with bf16 numerators in float64; the
    reference moves to a tile's maximum when that lies more than `lazy` above it."""
    m, l, o = -np.inf, 0.0, np.zeros(V.shape[1])
    for x, rows in tiles:
        if x.max() > m + lazy:
            l, o, m = l * np.exp2(m - x.max()), o * np.exp2(m - x.max()), x.max()
        p = np.exp2(x - m)
        l += p.sum()
        o += parity.to_f64(_bf16(p)) @ V[rows]
    return _bf16(o / l)


@pytest.mark.parametrize("form", ["single launch", "single launch, no stop rule", "no stop rule, no state"])
def test_reference_follows_the_running_maximum(gpu, form):
    """The bf16 rounding of the numerators falls at the scale of the reference, which moves when the
    maximum has grown by more than 2^8: here by 2^9.7 in the last tile of three.  The results are bf16
    values that float64 gives for that rule, but for the near-ties that fp32 sums can turn (1e-6 of
    a bf16 spacing of 2^-8 each: 0.1 %; the limit is 2 %), and not those of a reference that stays."""
    rng = np.random.default_rng(5)
    S, L, D = 64, 192, 128
    x = np.zeros(L)
    x[:S] = rng.integers(96, 155, S) / 16.0     # exact in bf16; all other keys have logit 0
    x[17] = 155 / 16.0
    K = np.zeros((L, D))
    K[:, 0] = x
    Q = np.zeros((L, D))
    Q[:, 0] = 1.0
    Vb = _bf16(rng.standard_normal((L, D)))
    V = parity.to_f64(Vb)
    scale = np.float32(np.log(2.0))
    logits = x * float(np.float32(scale * np.float32(1.4426950408889634)))
    non_causal = int(form == "no stop rule, no state")
    p = gu.s2o.make_params(1, 1, 1, L, D, S, 64, 64, use_q_perm=0, stop_mode=0 if form == "single launch" else 2,
                           softmax_scale=float(scale), non_causal=non_causal)
    first, second, own = np.arange(S), np.arange(S, 2 * S), np.arange(2 * S, L)     # segment 2 walks own, second, first
    kv = np.concatenate([own, second, first] * 3 if non_causal else [first, second, first]).astype(np.int32)
    dev = [gu.to_dev(b.reshape(1, 1, L, D)) for b in (_bf16(Q), _bf16(K), Vb)]
    kvd = gu.torch.from_numpy(kv.reshape(1, 1, -1)).to("cuda:0")
    print(f"case: {form}, L={L} S={S}, logits up to 2^9.7 above the first tile's", flush=True)
    O, _, _ = gu.s2o.s2o_attention(*dev, p, None, kvd, 0.0, two_pass=False)
    gu.torch.cuda.synchronize()
    got = gu.bits_of(O)[0, 0, 2 * S:]
    walks = [(own if non_causal else own[:i + 1], second, first) for i in range(S)]
    want, stays = (np.stack([_online([(logits[t], t) for t in w], V, lazy) for w in walks]) for lazy in (8.0, 16.0))
    assert (want != stays).mean() > 0.1
    assert (got != want).mean() <= 0.02, f"{(got != want).mean()} of the results differ"
