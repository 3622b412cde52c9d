"""Both experts' tiles in one launch: every tile choice, all tokens with one expert, rows and columns that fill no tile."""
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("share", [0.0, 0.4, 1.0])
@pytest.mark.parametrize("T,K,N", [
    (1, 32, 4), (37, 96, 100), (65, 128, 64), (200, 512, 192),                       # 32-row slices, each stage width
    (700, 96, 300), (1300, 256, 260),                                                # ... over many row tiles
    (2000, 96, 300), (1801, 256, 260), (1379, 768, 768),                             # 64-row slices, each stage width
    (9001, 96, 301), (9000, 768, 512), (8700, 2048, 320), (8450, 512, 4096),         # the three larger pairs
])
def test_moe_linear_against_separate_launches(sa, T, K, N, share):
    g = torch.Generator(device="cuda")
    g.manual_seed(T + K + N)
    x = torch.randn((T, K), generator=g, device="cuda")
    xq, xh = sa.sa_quantize_act_half(x, 127.0 / 4.0)
    w4 = torch.randint(0, 256, (N, K // 2), generator=g, device="cuda", dtype=torch.uint8)
    wh = (torch.randn((N, K), generator=g, device="cuda") / K**0.5).half()
    shift = torch.rand(T, generator=g, device="cuda") < share
    logits = torch.stack((torch.where(shift, -1.0, 1.0), torch.where(shift, 1.0, -1.0)), dim=1).contiguous()
    got = sa.sa_moe_linear(xq, xh, logits, w4, wh, 0.01)
    ref = sa.sa_moe_linear(xq, xh, logits, w4, wh, 0.01, variant=0)      # a launch for each expert
    assert torch.equal(got[shift], ref[shift])
    torch.testing.assert_close(got[~shift], ref[~shift], rtol=1e-4, atol=1e-4)
