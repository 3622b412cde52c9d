"""A layer whose MLP is one launch that normalises its rows itself (and, with prepared weights, makes them: the output projection),
and whose Q, K, V projection normalises its rows, against one whose LayerNorms and projections are launches of their own (the
vector-ALU variant of the Shift Linears: integers, so the same sums)."""
import pytest
import torch

pytestmark = pytest.mark.gpu


# every width, both heights of a workgroup's rows (128 of 128 and more columns from 16385 rows on), rows that fill no workgroup; 194 rows
# of 192 and 500 of 256 keep launches of their own
@pytest.mark.parametrize("B,N,H,E,hid", [
    (1, 1, 1, 64, 256), (3, 77, 2, 64, 512), (1, 333, 2, 128, 256), (2, 97, 3, 192, 512), (5, 1601, 3, 192, 768),
    (1, 500, 4, 256, 384), (1, 10241, 4, 256, 1024), (7, 2801, 4, 256, 512), (9, 3001, 2, 128, 640),
    (4, 3101, 3, 192, 256), (1, 1537, 2, 128, 256), (6, 2801, 3, 192, 256),
    (1, 10367, 3, 192, 256), (1, 10368, 3, 192, 256),                       # either side of where Q, K, V take the LayerNorm in
    (2, 1601, 3, 192, 384), (4, 4201, 3, 192, 640), (1, 4099, 4, 256, 384), (2, 8301, 4, 256, 640),     # odd numbers of hidden chunks
    (1, 33001, 4, 256, 512), (1, 42599, 4, 256, 512),                       # a second round of rows nearly empty, and less so
])
def test_normalised_rows_stay_on_the_chip(sa, B, N, H, E, hid):
    g = torch.Generator(device="cuda")
    g.manual_seed(N + hid)
    T = B * N
    x = torch.randn((T, E), generator=g, device="cuda")
    gamma1, beta1, gamma2, beta2 = (torch.randn(E, generator=g, device="cuda") for _ in range(4))
    w = [torch.randint(0, 256, s, generator=g, device="cuda", dtype=torch.uint8)
         for s in ((3 * E, E // 2), (E, E // 2), (hid, E // 2), (E, hid // 2))]
    proj = torch.randn((E // H, 64), generator=g, device="cuda")
    lut = torch.arange(-128, 128, device="cuda").clamp(min=0).to(torch.int8)
    y = []
    for variant in (0, 2, 3):
        if variant == 3:
            w = [sa.sa_shift_planes_prepare(t) for t in w]
        layer = sa.binding.Layer(B=B, N=N, H=H, nbits=64, E=E, hid=hid, attention=0, moe=0, shift_variant=variant, eps=1e-6,
                                 ln_inv_scale=32.0, qkv_scale=2.0**-12, attn_scale=(64.0 * N) ** -0.5, act_inv_scale=32.0,
                                 o_scale=2.0**-12, requant_scale=2.0**-11, out_scale=2.0**-12, x=x, gamma1=gamma1, beta1=beta1,
                                 gamma2=gamma2, beta2=beta2, wqkv=w[0], wo=w[1], proj=proj, w1=w[2], w2=w[3], lut=lut)
        y.append(layer.forward().clone())
    assert float((y[0] - x).abs().max()) > 0.0
    assert torch.equal(y[0], y[1]) and torch.equal(y[0], y[2])
