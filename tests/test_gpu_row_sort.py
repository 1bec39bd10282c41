"""The plan's row sort at the edges of its shapes: rows that just fill one LDS sort and rows one
query tile longer (2048, 6656 and 13312 keys), rows cut into ranges and scanned once per range,
rows dealt out to the ranges first, ranges that have to be cut again because of many equal
scores, and far-off scores.  The scores come from the plan itself, so the maps must equal the
stable argsort of them entry for entry."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

from paper_2602_22575_amd import inputs
import gpu_util as gu


def _check(w, Qb, Kb, rows, non_causal=0):
    print(f"case: row sort L={w.L} S={w.S} H={w.H} non_causal={non_causal}", flush=True)
    _, pg = gu.gpu_plan(w, gu.to_dev(Qb), gu.to_dev(Kb), non_causal=non_causal)
    assert np.array_equal(pg["q_perm"], np.argsort(-pg["s_q"], axis=-1, kind="stable"))
    for h in range(w.H):
        for n in rows:
            o, ln = (n * w.L, w.L) if non_causal else (w.S * n * (n - 1) // 2, n * w.S)
            sk = pg["s_k"][0, h, o:o + ln]
            assert np.array_equal(pg["kv_perm"][0, h, o:o + ln], np.argsort(-sk, kind="stable")), (h, n)


@pytest.mark.parametrize("L,S", [(2112, 64), (2176, 64), (6720, 64), (6784, 64), (13376, 64), (13440, 64),
                                 (16384, 8192), (24576, 512)])
def test_row_lengths_around_the_sort_capacities(gpu, L, S):
    w = inputs.workload("llama8k", L=L, S=S, H=2, Hkv=1, seed=L)
    Qb, Kb, _ = inputs.make_qkv(w)
    N = w.N
    _check(w, Qb, Kb, sorted({1, 2, N // 2, N - 2, N - 1} - {0}))


def test_non_causal_rows_cut_into_ranges(gpu):
    w = inputs.workload("llama8k", L=20480, S=2048, H=2, Hkv=1, seed=4)
    Qb, Kb, _ = inputs.make_qkv(w)
    _check(w, Qb, Kb, (0, 9), non_causal=1)


@pytest.mark.parametrize("kind", ["plain", "equal", "few values", "far-off"])
@pytest.mark.parametrize("H", [1, 9])
def test_long_rows(gpu, H, kind):
    """32K tokens in 128 segments: one head is scanned per range, nine heads (1143 rows) are dealt
    out.  Equal scores overflow ranges and regions; a far-off score stretches the range."""
    w = inputs.workload("llama8k", L=32768, S=256, H=H, Hkv=1, seed=7)
    Qb, Kb, _ = inputs.make_qkv(w)
    if kind == "equal":
        Kb[0, 0, 3000:25000] = Kb[0, 0, 3000]
    elif kind == "few values":
        Kb[:] = Kb[0, 0, 7]
        Kb[0, 0, ::3, 0] ^= 0x8000
    elif kind == "far-off":
        K = inputs.bf16_bits_to_f32(Kb)
        K[0, 0, 5] *= 1000
        K[0, 0, -300] *= -3000
        Kb = inputs.f32_to_bf16_bits(K)
    _check(w, Qb, Kb, (1, 26, 27, 100, 126, 127) if H == 1 else (60, 127))


@pytest.mark.parametrize("kind", ["nan query", "nan keys", "nan and infinite keys"])
@pytest.mark.parametrize("H", [1, 9])
def test_long_rows_with_nan(gpu, H, kind):
    """NaN scores are an input error, but every row of the maps stays a permutation, also where all
    scores of a row are NaN (one NaN in a query) and where infinities stand beside them; the other
    queries of such a segment attend as ever (here: without skipping, so densely)."""
    w = inputs.workload("llama8k", L=32768, S=256, H=H, Hkv=1, seed=8)
    Qb, Kb, Vb = inputs.make_qkv(w)
    n = 120
    bad = n * w.S + 77
    if kind == "nan query":
        Qb[0, H // 2, bad, 3] = 0x7fc0
    else:
        Kb[0, 0, 3000:3005, 9] = 0x7fc0
    if kind == "nan and infinite keys":
        Q = inputs.bf16_bits_to_f32(Qb)
        Qb = inputs.f32_to_bf16_bits(Q + 0.5)                 # every mean is about 0.5, 128 of them times 3e38 overflow
        Kb[0, 0, 4000:4100] = 0x7f61
        Kb[0, 0, 5000:5100] = 0xff61
    Qd, Kd, Vd = (gu.to_dev(x) for x in (Qb, Kb, Vb))
    print(f"case: row sort with {kind}, L={w.L} S={w.S} H={H}", flush=True)
    p = gu.params_for(w)
    maps = (gu.torch.full((1, H, w.N, w.S), -1, dtype=gu.torch.int32, device="cuda:0"),
            gu.torch.full((1, H, w.S * w.N * (w.N - 1) // 2), -1, dtype=gu.torch.int32, device="cuda:0"))
    plan = gu.s2o.s2o_plan(Qd, Kd, p, want_scores=True, maps=maps)
    gu.torch.cuda.synchronize()
    assert int(plan.status.item()) == 0
    sk, kv = plan.s_k.cpu().numpy()[0], plan.kv_perm.cpu().numpy()[0]
    assert np.isnan(sk).any() and np.isinf(sk).any() == (kind == "nan and infinite keys")
    for row in range(1, w.N):
        o, ln = w.S * row * (row - 1) // 2, row * w.S
        assert np.array_equal(np.sort(kv[:, o:o + ln], axis=1), np.broadcast_to(np.arange(ln), (H, ln))), row
    for row in (20, n, w.N - 1):                              # NaN is taken for -inf
        o, ln = w.S * row * (row - 1) // 2, row * w.S
        s = np.where(np.isnan(sk[:, o:o + ln]), -np.inf, sk[:, o:o + ln])
        assert np.array_equal(kv[:, o:o + ln], np.argsort(-s, axis=1, kind="stable")), row
    if kind == "nan query":
        Ob, c, s = gu.gpu_attention(w, Qd, Kd, Vd, plan.q_perm, plan.kv_perm, 0.0)
        h, rows = H // 2, np.array([0, 76, 78, 255]) + n * w.S
        f64 = [inputs.bf16_bits_to_f32(x).astype(np.float64) for x in (Qb[0, h, rows], Kb[0, 0], Vb[0, 0])]
        x = f64[0] @ f64[1].T / np.sqrt(w.D)
        x[np.arange(w.L)[None, :] > rows[:, None]] = -np.inf
        e = np.exp(x - x.max(axis=1, keepdims=True))
        ref = (e / e.sum(axis=1, keepdims=True)) @ f64[2]
        assert np.abs(inputs.bf16_bits_to_f32(Ob)[0, h, rows] - ref).max() <= 2e-2


@pytest.mark.parametrize("kind", ["tiny", "infinite"])
@pytest.mark.parametrize("L,S", [(2112, 64), (6720, 64), (13376, 64), (32768, 2048)])
def test_extreme_score_ranges(gpu, L, S, kind):
    """Scores whose range is denormal (its reciprocal infinite) or infinite: the map from score to
    bucket has to stay inside the buckets and monotone."""
    w = inputs.workload("llama8k", L=L, S=S, H=2, Hkv=1, seed=L)
    Qb, Kb, _ = inputs.make_qkv(w)
    K = inputs.bf16_bits_to_f32(Kb)
    Q = inputs.bf16_bits_to_f32(Qb)
    if kind == "tiny":
        Q, K = np.zeros_like(Q), np.zeros_like(K)
        Q[..., 0] = 2.0 ** -70
        K[..., 0] = 2.0 ** -76 * np.random.default_rng(1).integers(0, 8, L)[None, None, :]
        K[0, 0, 40] *= -1
    else:
        Q += 0.5
        K[0, 0, S:S + 3] = 3e38
        K[0, 0, 2 * S - 5:2 * S] = -3e38
    _check(w, inputs.f32_to_bf16_bits(Q), inputs.f32_to_bf16_bits(K), sorted({1, 2, w.N // 2, w.N - 1}))
