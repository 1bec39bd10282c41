"""The own-segment pass with one and with two row blocks a workgroup, and the order its workgroups come in: every
row's state is there, and a (batch, KV head)'s has the bits of the same heads on their own."""
import pytest

pytestmark = pytest.mark.gpu

import gpu_util as gu

# Z, H, Hkv, N, S, token-major
CASES = [
    (1, 3, 1, 7, 128, 0),            # a single block a segment
    (2, 6, 2, 5, 256, 1),            # one block each, longest first: all in flight at once
    (1, 12, 4, 33, 256, 0),          # pairs: 396 nearly fill a round
    (1, 18, 6, 32, 192, 1),          # one block each, unit by unit: 576 pairs, half a last block
    (1, 12, 4, 33, 320, 0),          # longest first: 792 pairs, an odd number of blocks, 132 units
    (1, 12, 4, 32, 320, 0),          # unit by unit: 768 pairs, 128 units
    (2, 9, 3, 29, 320, 1),           # pairs: 1044, a batch, strides, 174 units
    (1, 10, 2, 22, 512, 0),          # longest first: 440 pairs, 44 units
    (1, 10, 2, 24, 512, 0),          # unit by unit: 480 pairs, 48 units
    (1, 10, 5, 50, 512, 0),          # longest first: 1000 pairs, 250 units
    (3, 5, 1, 9, 1088, 1),           # longest first: 675 pairs, 9 blocks a segment, 27 units
    (1, 7, 7, 23, 1920, 0),          # longest first: 1288 pairs, 15 blocks
    (1, 8, 2, 16, 1024, 0),          # unit by unit: 512 pairs, 32 units
    (1, 16, 4, 24, 1024, 1),         # pairs: 1536, 96 units
    (1, 8, 2, 41, 1152, 1),          # pairs: 1640, 82 units
]


def _states(q, k, v, S, token):
    """(accumulator, l, m) per (z, head), the buffer filled with NaN before."""
    torch = gu.torch
    (Z, H, L, D), Hkv = q.shape, k.shape[1]
    strides = {}
    if token:
        q, k, v = (x.transpose(1, 2).contiguous() for x in (q, k, v))
        strides = dict(q_stride=(L * H * D, D, H * D), k_stride=(L * Hkv * D, D, Hkv * D), v_stride=(L * Hkv * D, D, Hkv * D))
    else:
        q, k, v = (x.contiguous() for x in (q, k, v))
    p = gu.s2o.make_params(Z, H, Hkv, L, D, S, 64, 64, **strides)
    state = torch.full((gu.s2o.s2o_attention_sizes(p)["scratch"],), 0xff, dtype=torch.uint8, device=q.device)
    st = gu.s2o.s2o_attention_local(q, k, v, p, scratch=state).view(torch.float32)
    rows = Z * H * L
    return [st[a * rows:b * rows].view(Z, H, -1) for a, b in ((0, D), (D, D + 1), (D + 1, D + 2))]


@pytest.mark.parametrize("Z,H,Hkv,N,S,token", CASES)
def test_state_among_others_and_alone(gpu, Z, H, Hkv, N, S, token):
    torch = gu.torch
    L, G = N * S, H // Hkv
    g = torch.Generator(device="cuda:0")
    g.manual_seed(S + N)
    q, k, v = (torch.randn((Z, h, L, 128), generator=g, device="cuda:0").to(torch.bfloat16) for h in (H, Hkv, Hkv))
    print(f"case: Z={Z} H={H} Hkv={Hkv} N={N} S={S} token-major={token}", flush=True)
    whole = _states(q, k, v, S, token)
    assert all(bool(torch.isfinite(x).all()) for x in whole)
    for z in range(Z):
        for i in range(Hkv):
            part = _states(q[z:z + 1, i * G:i * G + G], k[z:z + 1, i:i + 1], v[z:z + 1, i:i + 1], S, 0)
            for a, b in zip(whole, part):
                assert torch.equal(a[z, i * G:i * G + G], b[0]), (z, i)
