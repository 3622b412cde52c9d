"""The experts' hidden rows in columns of 64 bytes, against a launch for each expert, whose hidden rows are whole."""
import pytest
import torch

pytestmark = pytest.mark.gpu


# 64 x 64 tiles beyond the small tiles' range, rows that fill no tile, the shortest hidden rows of the rule and ragged longer ones
@pytest.mark.parametrize("share", [0.0, 0.5, 1.0])
@pytest.mark.parametrize("B,N,H,hid", [(18, 197, 12, 2048), (10, 821, 5, 2176), (1, 7001, 6, 2304)])
def test_block_against_separate_launches(sa, B, N, H, hid, share):
    g = torch.Generator(device="cuda")
    g.manual_seed(N + hid)
    T, E = B * N, H * 64
    q, k, v = (torch.randn((B, N, H, 64), generator=g, device="cuda") for _ in range(3))
    proj = torch.randn((64, 64), generator=g, device="cuda")
    shift = torch.rand(T, generator=g, device="cuda") < share
    logits = torch.stack((torch.where(shift, -1.0, 1.0), torch.where(shift, 1.0, -1.0)), dim=1).contiguous()
    w1, w2 = (torch.randint(0, 256, s, generator=g, device="cuda", dtype=torch.uint8) for s in ((hid, E // 2), (E, hid // 2)))
    lut = torch.arange(-128, 128, device="cuda").clamp(min=0).to(torch.int8)
    mw1 = (torch.randn((hid, E), generator=g, device="cuda") / E**0.5).half()
    mw2 = (torch.randn((E, hid), generator=g, device="cuda") / hid**0.5).half()
    y = []
    for variant in (2, 0):
        b = sa.binding.Block(B=B, N=N, H=H, d=64, nbits=64, dv=64, attention=0, hid=hid, moe=True, attn_scale=(64 * N) ** -0.5,
                             act_inv_scale=32.0, requant_scale=2.0**-12, out_scale=2.0**-12, q=q, k=k, v=v, proj=proj,
                             logits=logits, w1=w1, w2=w2, lut=lut, mw1=mw1, mw2=mw2, shift_variant=variant)
        b.forward()
        y.append(b.y)
    assert float(y[0].abs().max()) > 0.0
    assert torch.equal(y[0][shift], y[1][shift])
    torch.testing.assert_close(y[0][~shift], y[1][~shift], rtol=1e-4, atol=1e-4)
