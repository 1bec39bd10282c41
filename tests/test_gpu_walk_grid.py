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
