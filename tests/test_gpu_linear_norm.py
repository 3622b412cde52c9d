"""A layer whose output projection, residual and second LayerNorm are one launch (prepared weights), against the same layer on packed
weights, whose are two: the same integer sums, the same order of the row's sums, so the same bits."""
import pytest
import torch

pytestmark = pytest.mark.gpu


# every width; one row, either side of a workgroup's 16, the last row count that takes it and one more; with and without a router
@pytest.mark.parametrize("moe", [True, False])
@pytest.mark.parametrize("T,E,H", [(1, 64, 1), (15, 128, 2), (16, 192, 3), (17, 64, 2), (33, 192, 3), (1000, 128, 4), (2000, 192, 6),
                                   (32768, 64, 1), (32769, 64, 1), (16384, 128, 2), (16385, 128, 2), (10922, 192, 3), (10923, 192, 3)])
def test_projection_and_norm_in_one_launch(sa, T, E, H, moe):
    g = torch.Generator(device="cuda")
    g.manual_seed(T + E)
    hid = 4 * E + 64                                         # (no MLP in one launch with the projection in it)
    x = torch.randn((T, E), generator=g, device="cuda")
    x[T // 2] = float("nan") if T > 2 else 0.25
    gamma1, beta1, gamma2, beta2 = (torch.randn(E, generator=g, device="cuda") for _ in range(4))
    w = [torch.randint(0, 256, s, generator=g, device="cuda", dtype=torch.uint8)
         for s in ((3 * E, E // 2), (E, E // 2), (hid, E // 2), (E, hid // 2))]
    kw = {}
    if moe:
        kw = dict(wg=torch.randn((E, 2), generator=g, device="cuda"), bg=torch.randn(2, generator=g, device="cuda"),
                  mw1=torch.randn((hid, E), generator=g, device="cuda").half() * 0.1, mw2=torch.randn((E, hid), generator=g, device="cuda").half() * 0.1)
    proj = torch.randn((E // H, 64), generator=g, device="cuda")
    lut = torch.arange(-128, 128, device="cuda").clamp(min=0).to(torch.int8)
    y = []
    for variant in (2, 3):
        if variant == 3:
            w = [sa.sa_shift_planes_prepare(t) for t in w]
        layer = sa.binding.Layer(B=1, N=T, H=H, nbits=64, E=E, hid=hid, attention=0, moe=int(moe), shift_variant=variant, eps=1e-6,
                                 ln_inv_scale=32.0, qkv_scale=2.0**-12, attn_scale=(64.0 * T) ** -0.5, act_inv_scale=32.0, o_scale=2.0**-12,
                                 requant_scale=2.0**-11, out_scale=2.0**-12, x=x, gamma1=gamma1, beta1=beta1, gamma2=gamma2, beta2=beta2,
                                 wqkv=w[0], wo=w[1], proj=proj, w1=w[2], w2=w[3], lut=lut, **kw)
        y.append(layer.forward().clone())
    rows = torch.isfinite(x).all(dim=1)
    assert float((y[0] - x)[rows].abs().max()) > 0.0
    assert torch.equal(y[0].nan_to_num(nan=3.0), y[1].nan_to_num(nan=3.0))
