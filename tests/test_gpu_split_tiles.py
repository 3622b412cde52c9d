"""Launches of both experts whose last rows go to lower tiles: routings on either side of where that fills the last round of workgroups, all
tokens with one expert, row counts that are no whole tiles, as Linears and as both layers of a block, whose hidden rows are in columns, against a
launch for each expert."""
import pytest
import torch

from test_gpu_hidden_columns import test_block_against_separate_launches as block_against_separate_launches

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T,K,N,share", [
    (12608, 768, 3072, 0.70), (12608, 768, 3072, 0.62), (12608, 768, 3072, 0.0), (12608, 768, 3072, 1.0), (13001, 768, 3072, 0.45),      # Mult rows
    (12608, 3072, 768, 0.70), (12608, 3072, 768, 0.55), (12608, 3072, 768, 1.0), (11777, 2048, 640, 0.80), (10001, 3072, 768, 0.97),     # Shift rows
    (28001, 768, 3072, 0.50), (14001, 3072, 768, 0.55),              # beyond the last round that takes lower tiles
])
def test_lower_tiles_for_the_last_rows(sa, T, K, N, share):
    g = torch.Generator(device="cuda")
    g.manual_seed(T + K + int(100 * share))
    x = torch.randn((T, K), generator=g, device="cuda")
    xq, xh = sa.sa_quantize_act_half(x, 127.0 / 4.0)
    w4 = torch.randint(0, 256, (N, K // 2), generator=g, device="cuda", dtype=torch.uint8)
    wh = (torch.randn((N, K), generator=g, device="cuda") / K**0.5).half()
    shift = torch.rand(T, generator=g, device="cuda") < share
    logits = torch.stack((torch.where(shift, -1.0, 1.0), torch.where(shift, 1.0, -1.0)), dim=1).contiguous()
    y = torch.full((T, N), float("nan"), device="cuda")
    got = sa.sa_moe_linear(xq, xh, logits, w4, wh, 0.01, y=y)
    ref = sa.sa_moe_linear(xq, xh, logits, w4, wh, 0.01, variant=0)
    assert torch.equal(got[shift], ref[shift])
    # fp32 sums of K products in two orders: a partial sum, of rms up to 1, is rounded K / 16 times (half of 2^-23 at most, 2^-24 rms): 3072 / 16 of
    # these are 200 * 2^-24 = 1.2e-5 at worst on either side, as test_gpu_experts.py allows
    torch.testing.assert_close(got[~shift], ref[~shift], rtol=1e-4, atol=1e-4)


@pytest.mark.parametrize("share", [0.0, 0.45, 0.55, 0.62, 0.70, 0.97])
@pytest.mark.parametrize("B,N,H,hid", [(64, 197, 12, 3072), (1, 10001, 12, 3072)])
def test_block(sa, B, N, H, hid, share):
    block_against_separate_launches(sa, B, N, H, hid, share)
