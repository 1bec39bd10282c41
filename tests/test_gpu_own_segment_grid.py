"""The own-segment pass with one and with two row blocks a workgroup: the state of a head among 1024 pairs
of blocks or fewer, and among more, is the same, bit for bit, over segments of one block, of an odd and of an
even number of blocks, and of a block that is only half full."""
import pytest

pytestmark = pytest.mark.gpu

import gpu_util as gu


@pytest.mark.parametrize("S", [64, 128, 192, 320, 512])
def test_state_with_single_and_paired_blocks(gpu, S):
    torch = gu.torch
    pairs = ((S + 127) // 128 + 1) // 2
    N = 8
    H = 1024 // (N * pairs)                        # at most 1024 pairs; one head more: above
    g = torch.Generator(device="cuda:0")
    g.manual_seed(S)
    q, k, v = (torch.randn((1, H + 1, N * S, 128), generator=g, device="cuda:0").to(torch.bfloat16) for _ in range(3))
    out = []
    for h in (H, H + 1):
        print(f"case: S={S} heads={h} pairs={h * N * pairs}", flush=True)
        p = gu.s2o.make_params(1, h, h, N * S, 128, S, 64, 64)
        st = gu.s2o.s2o_attention_local(*(x[:, :h].contiguous() for x in (q, k, v)), p).view(torch.float32)
        rows = h * N * S
        out.append((st[:rows * 128].view(h, -1), st[rows * 128:rows * 129].view(h, -1), st[rows * 129:rows * 130].view(h, -1)))
    for a, b in zip(*out):
        assert torch.equal(a, b[:H]) and bool(torch.isfinite(b).all())
