"""Which rankings deal long rows out to score ranges (split) instead of scanning a row once per range,
on both sides of the rule's lines, and that both ways rank alike."""
import pytest

from paper_2602_22575_amd import binding as b

CAP, GROUPS = 6656, 512                 # keys of the sort that long rows use; workgroups that split


def _ranges(length):
    return -(-length // (CAP - 7 * (CAP // 25)))


# (H, L, S, non_causal, split)
SHAPES = [
    (1, 131072, 512, 0, False),         # 255 rows of 28 ranges
    (2, 131072, 512, 0, False),         # 510
    (3, 131072, 512, 0, True),          # 765
    (3, 65536, 256, 0, False),          # 765 rows of 14 ranges
    (4, 65536, 256, 0, True),           # 1020
    (5, 65536, 4096, 1, False),         # 80 rows of 15 ranges
    (8, 65536, 2048, 1, False),         # 256
    (12, 65536, 2048, 1, False),        # 384
    (13, 65536, 2048, 1, True),         # 416
    (17, 65536, 2048, 1, False),        # 544: a second round on 512 workgroups
    (24, 65536, 2048, 1, True),         # 768
    (16, 32768, 1024, 1, False),        # 512 rows of 8 ranges: the scans are short
]


@pytest.mark.parametrize("H,L,S,nc,split", SHAPES)
def test_side_of_the_rule(H, L, S, nc, split):
    """A split ranking needs the score array and the ranges' regions of every splitting workgroup."""
    N = L // S
    rows, keys = H * (N if nc else N - 1), H * (N * L if nc else S * N * (N - 1) // 2)
    regions = min(rows, GROUPS) * _ranges(L if nc else L - S) * CAP * 8
    scratch = b.s2o_plan_sizes(b.make_params(1, H, 1, L, 128, S, non_causal=nc))["scratch"]
    assert (scratch >= 4 * keys + regions) == split, (scratch, 4 * keys, regions)
    assert scratch <= max(8 * keys, 4 * keys + regions) + 64 * rows * 32 + rows * L // 8 + (1 << 21)


@pytest.mark.gpu
@pytest.mark.parametrize("H,L,S,nc,split", [s for s in SHAPES if s[0] * s[1] * s[1] // s[2] <= 200e6])
def test_rows_on_both_sides(gpu, H, L, S, nc, split):
    import torch
    import paper_2602_22575_amd as s2o
    g = torch.Generator(device="cuda:0")
    g.manual_seed(L + H)
    Q, K = (torch.randn((1, h, L, 128), generator=g, device="cuda:0") for h in (H, 1))
    Q += 0.25                                                     # far-off scores for a few keys
    K[:, :, ::1013] += 0.5
    K[0, 0, L // 3:L // 3 + L // 16] = K[0, 0, L // 3].clone()    # equal scores: some ranges hold more than a sort
    print(f"case: H={H} L={L} S={S} non_causal={nc} split={split}", flush=True)
    plan = s2o.s2o_plan(Q.bfloat16(), K.bfloat16(), s2o.make_params(1, H, 1, L, 128, S, non_causal=nc), want_scores=True)
    torch.cuda.synchronize()
    assert int(plan.status.item()) == 0
    kv, sk = plan.kv_perm.view(H, -1), plan.s_k.view(H, -1)
    for n in range(0 if nc else 1, L // S):
        o, ln = (n * L, L) if nc else (S * n * (n - 1) // 2, n * S)
        want = torch.sort(sk[:, o:o + ln], dim=1, descending=True, stable=True).indices
        assert torch.equal(kv[:, o:o + ln].long(), want), n
