"""s_Q, q_mean and Q_perm of segments that take the larger shapes of the query sort, at the edges of
these shapes (2048, 6656 and 8192 queries; 16-row groups that end inside a trip of the pooling loop)."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

from paper_2602_22575_amd import inputs
import gpu_util as gu


@pytest.mark.parametrize("kind", ["gaussian", "few values", "far-off"])
@pytest.mark.parametrize("S", [2048, 2112, 5632, 6656, 6720, 8192])
def test_long_segments(gpu, S, kind):
    w = inputs.workload("llama8k", L=2 * S, S=S, H=3, Hkv=1, seed=S)
    Qb, Kb, _ = inputs.make_qkv(w)
    Q = inputs.bf16_bits_to_f32(Qb)
    if kind == "few values":                            # 40 rows over and over: every bucket is crowded
        Q = Q[:, :, np.arange(w.L) % 40]
    elif kind == "far-off":
        Q[0, 1, S + 5:S + 400] *= 1000
        Q[0, 2, 7] *= -3000
    Qb = inputs.f32_to_bf16_bits(Q)
    print(f"case: query sort S={S} {kind}", flush=True)
    _, pg = gu.gpu_plan(w, gu.to_dev(Qb), gu.to_dev(Kb))
    assert np.array_equal(pg["q_perm"], np.argsort(-pg["s_q"], axis=-1, kind="stable"))
    Q = inputs.bf16_bits_to_f32(Qb).astype(np.float64).reshape(1, w.H, w.N, S, w.D)
    # a sum of n fp32 terms is off by at most n * 2^-24 of the sum of their absolute values: S/16 terms
    # in a row and a tree over the rest for the means, 8 and a tree of 16 for the dot products (k_guide's
    # own rounding counts through kg, which is taken from the device)
    mean, room = Q.mean(axis=3), np.abs(Q).mean(axis=3) * ((S // 16 + 8) * 2.0 ** -24)
    assert np.all(np.abs(pg["q_mean"] - mean) <= room)
    kg = pg["k_guide"][0, 0].astype(np.float64)
    assert np.all(np.abs(pg["s_q"] - Q @ kg) <= (np.abs(Q) @ np.abs(kg)) * (16 * 2.0 ** -24))


@pytest.mark.parametrize("S,L", [(64, 128), (576, 1152), (1024, 32768), (2112, 4224), (8192, 16384)])
def test_scores_come_back_as_they_are(gpu, S, L):
    """A query that is not a number: its score comes back as one while the sort takes it for the lowest."""
    w = inputs.workload("llama8k", L=L, S=S, H=3, Hkv=1, seed=S)
    Qb, Kb, _ = inputs.make_qkv(w)
    Q = inputs.bf16_bits_to_f32(Qb)
    bad = (0, S - 1, S // 2 + 3)
    for i in bad:
        Q[0, 1, S + i, 5] = np.nan
    print(f"case: NaN queries S={S} L={L}", flush=True)
    out = gu.s2o.s2o_plan(gu.to_dev(inputs.f32_to_bf16_bits(Q)), gu.to_dev(Kb), gu.params_for(w), want_scores=True)
    gu.torch.cuda.synchronize()
    sq, perm = out.s_q.cpu().numpy(), out.q_perm.cpu().numpy()
    where = np.zeros(sq.shape, bool)
    where[0, 1, 1, list(bad)] = True
    assert np.array_equal(np.isnan(sq), where)
    assert np.array_equal(perm, np.argsort(-np.where(where, -np.inf, sq), axis=-1, kind="stable"))
