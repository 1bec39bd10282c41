"""A threshold of 0 or less takes the walk without votes: the bits and the counts of the walk with votes
at a threshold so small that no tile's mass lies below it, over orders, tile heights, modes and maps,
also where the logits grow from tile to tile and the softmax reference moves."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

from paper_2602_22575_amd import inputs
import gpu_util as gu

TINY = 1e-37            # below the mass of a tile (at least 2^-100 of the sum here) but not a threshold of 0


@pytest.mark.parametrize("scale", [1.0, 6.0])
@pytest.mark.parametrize("non_causal,mapped", [(0, True), (1, True), (1, False)])
@pytest.mark.parametrize("L,S,BM", [(128, 64, 64), (704, 64, 64), (1920, 640, 128), (4096, 512, 64)])
def test_same_bits_without_votes(gpu, L, S, BM, non_causal, mapped, scale):
    w = inputs.workload("llama8k", L=L, S=S, H=4, Hkv=2, seed=L + S)
    Qb, Kb, Vb = inputs.make_qkv(w)
    ramp = np.linspace(1.0, scale, L)[::-1] if mapped else np.linspace(1.0, scale, L)
    Kb = inputs.f32_to_bf16_bits((inputs.bf16_bits_to_f32(Kb) * ramp[None, None, :, None]).astype(np.float32))
    Q, K, V = (gu.to_dev(x) for x in (Qb, Kb, Vb))
    for q_perm in (0, 1):
        for mode in (0, 1):
            p = gu.s2o.make_params(1, 4, 2, L, 128, S, BM, 64, use_q_perm=q_perm, stop_mode=mode, non_causal=non_causal)
            plan = gu.s2o.s2o_plan(Q, K, p, want_scores=False)
            kv = plan.kv_perm if mapped else None
            print(f"case: L={L} S={S} BM={BM} non_causal={non_causal} mapped={mapped} q_perm={q_perm} mode={mode}", flush=True)
            votes = gu.s2o.s2o_attention(Q, K, V, p, plan.q_perm, kv, TINY)
            n_tiles = np.repeat([L // 64 if non_causal else n * S // 64 for n in range(L // S)], S // BM)
            assert np.all(votes[1].cpu().numpy() == n_tiles) and not votes[2].cpu().numpy().any()
            for tau in (0.0, -0.0, -1.0):
                got = gu.s2o.s2o_attention(Q, K, V, p, plan.q_perm, kv, tau)
                assert np.array_equal(gu.bits_of(got[0]), gu.bits_of(votes[0]))
                assert all(gu.torch.equal(a, b) for a, b in zip(got[1:], votes[1:]))
