"""The ranking of few segments (query sort beside the scores) against the ranking of the same
sequences inside a larger batch (query sort in front of the scores): both add in the same order, so
every output is the same, bit for bit."""
import pytest

from paper_2602_22575_amd import binding as b

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("L,S,H,Hkv,Z", [
    (64, 64, 1, 1, 385),        # one segment: nothing to score
    (576, 64, 5, 1, 9),         # an odd number of rows; 45 beside, 405 in front
    (2560, 512, 4, 2, 20),      # the largest segment of the smaller sort; 20 beside, 400 in front
    (1152, 576, 4, 4, 49),      # the smallest of the larger sort; 8 and 392
    (3072, 64, 8, 2, 2),        # exactly the limit on the rows, then twice that
    (1024, 256, 4, 2, 20),      # 16 rows, then 320: over the lower limit on the queries from 257 rows on
    (4096, 2048, 32, 8, 2),     # 64 rows of 2048: exactly the limit on the queries, then twice that
])
def test_both_places_of_the_query_sort(gpu, L, S, H, Hkv, Z):
    import torch
    gen = torch.Generator(device="cuda:0")
    gen.manual_seed(L + S)
    Q = torch.randn((Z, H, L, 128), generator=gen, device="cuda:0").to(torch.bfloat16)
    K = torch.randn((Z, Hkv, L, 128), generator=gen, device="cuda:0").to(torch.bfloat16)
    print(f"case: L={L} S={S} H={H} Hkv={Hkv} batch {Z}", flush=True)
    all_ = b.s2o_plan(Q, K, b.make_params(Z, H, Hkv, L, 128, S))
    for z in (0, Z - 1):
        one = b.s2o_plan(Q[z:z + 1].contiguous(), K[z:z + 1].contiguous(), b.make_params(1, H, Hkv, L, 128, S))
        torch.cuda.synchronize()
        assert int(all_.status.item()) == 0 and int(one.status.item()) == 0
        for name in ("q_perm", "s_q", "q_mean", "k_guide") + (("kv_perm", "s_k") if L > S else ()):
            got, ref = getattr(one, name), getattr(all_, name)[z:z + 1]
            assert got.shape == ref.shape and torch.equal(got.view(torch.int32), ref.view(torch.int32)), (name, z)
