"""The walk's block ids: every (head, segment, query tile) is taken once, whatever the number of heads
(a multiple of 8 or not) and of workgroups a segment has (a full run of 4, a remainder, a single one,
more runs than XCDs).  A head's results depend on its own inputs alone, so those of H heads have to
be the bits of the same heads among 8."""
import pytest

pytestmark = pytest.mark.gpu

from paper_2602_22575_amd import inputs
import gpu_util as gu


@pytest.mark.parametrize("H", [1, 3, 5])
@pytest.mark.parametrize("L,S,BM", [(192, 64, 64), (1152, 384, 128), (1920, 640, 64), (1152, 576, 64), (2304, 1152, 64),
                                    (4224, 4224, 64)])
def test_heads_alone_and_among_eight(gpu, H, L, S, BM):
    w = inputs.workload("llama8k", L=L, S=S, H=8, Hkv=8, seed=L + S)
    Q, K, V = (gu.to_dev(x) for x in inputs.make_qkv(w))
    torch = gu.torch
    for tau in (0.0, 0.05):
        for two_pass in (True, False):
            print(f"case: H={H} L={L} S={S} BM={BM} tau={tau} two_pass={two_pass}", flush=True)
            out = []
            for h in (8, H):
                q, k, v = (x[:, :h].contiguous() for x in (Q, K, V))
                p = gu.s2o.make_params(1, h, h, L, 128, S, BM, 64)
                plan = gu.s2o.s2o_plan(q, k, p, want_scores=False)
                O = torch.full_like(q, float("nan"))
                counts = [torch.full((1, h, L // BM), -1, dtype=torch.int32, device=q.device) for _ in range(2)]
                gu.s2o.s2o_attention(q, k, v, p, plan.q_perm, plan.kv_perm, tau, O=O, computed=counts[0],
                                     skipped=counts[1], two_pass=two_pass)
                out.append([O, *counts])
            for a, b in zip(*out):
                assert torch.equal(gu.torch.nan_to_num(a[:, :H].float(), nan=7e7), gu.torch.nan_to_num(b.float(), nan=7e7))
            assert not torch.isnan(out[1][0].float()).any() and all((c >= 0).all() for c in out[1][1:])


@pytest.mark.parametrize("H,N,S,mapped", [
    (12, 1, 5248, 0),        # runs of 3 where 4 would overfill an XCD
    (6, 1, 5248, 1),         # of 2
    (5, 1, 6528, 0),         # one by one
    (12, 1, 2048, 1),        # of 4
    (9, 1, 7296, 0),         # of 4, with a remainder
    (4, 4, 1280, 1),         # of 4 and 2 in turn
])
def test_runs_without_causality(gpu, H, N, S, mapped):
    """Where all walks have one length the runs are shorter if they would overfill an XCD: every query tile is
    still taken once, with the bits it has among 8 or 16 heads (one segment's heads in turn, no runs)."""
    L, among = N * S, 8 if H < 8 else 16
    w = inputs.workload("llama8k", L=L, S=S, H=among, Hkv=among, seed=S)
    Q, K, V = (gu.to_dev(x) for x in inputs.make_qkv(w))
    torch = gu.torch
    print(f"case: H={H} N={N} S={S} mapped={mapped}", flush=True)
    out = []
    for h in (among, H):
        q, k, v = (x[:, :h].contiguous() for x in (Q, K, V))
        p = gu.s2o.make_params(1, h, h, L, 128, S, 64, 64, stop_mode=2, non_causal=1, use_q_perm=mapped, max_prefix_tiles=7)
        maps = (None, None)
        if mapped:
            plan = gu.s2o.s2o_plan(q, k, p, want_scores=False)
            maps = (plan.q_perm, plan.kv_perm)
        O = torch.full_like(q, float("nan"))
        counts = [torch.full((1, h, L // 64), -1, dtype=torch.int32, device=q.device) for _ in range(2)]
        gu.s2o.s2o_attention(q, k, v, p, *maps, 0.0, O=O, computed=counts[0], skipped=counts[1])
        out.append([O, *counts])
    for a, b in zip(*out):
        assert torch.equal(a[:, :H], b) and not torch.isnan(b.float()).any()
    assert all(bool((c >= 0).all()) for c in out[1][1:])
