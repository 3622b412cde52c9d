"""The matrix-core hash against its defining fp32 chain where the fp16 terms, the margin or the split of the work can go wrong:
every number of hash columns per workgroup, rows that do not fill a tile, magnitudes outside what splits unscaled, rows and
columns that settle every bit by the chain."""
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kind", ["plain", "scales", "degenerate"])
@pytest.mark.parametrize("d,nbits", [(32, 64), (32, 128), (32, 256), (64, 64), (64, 128), (64, 192), (64, 256), (64, 512),
                                     (128, 64), (128, 128), (128, 256)])
@pytest.mark.parametrize("B,N,H", [(1, 1, 1), (2, 33, 3), (3, 1000, 4)])
def test_bits_are_the_chains(sa, B, N, H, d, nbits, kind):
    g = torch.Generator(device="cuda")
    g.manual_seed(d + nbits + N)
    x = [torch.randn((B, N, H, d), generator=g, device="cuda") for _ in range(2)]
    proj = torch.randn((d, nbits), generator=g, device="cuda")
    if kind == "scales":                                   # 2^-40 .. 2^40, some rows in denormal range
        for t in x:
            t *= torch.exp2(torch.randint(-40, 41, (B, N, H, 1), generator=g, device="cuda").float())
        x[0][:, ::7] *= 1e-38
        proj[:, ::5] *= 1e-6
    if kind == "degenerate":
        x[0][:, ::3] = 0.0
        x[1][:, ::5, :, 1] = float("inf")
        x[1][:, ::4, :, 0] = float("nan")
        x[0][:, 1::2, :, 2:] = 0.0                         # sums of two products: cancellation is common
        proj[:, 1::9] = 0.0
        proj[0, ::11] = 1e30
    codes = [torch.zeros((B, H, N, nbits // 64), dtype=torch.int64, device="cuda") for _ in range(2)]
    sa.sa_binarize_pair(x[0], x[1], proj, nbits, codes[0], codes[1])
    for t, c in zip(x, codes):
        assert torch.equal(c, sa.sa_binarize(t, proj, nbits, variant=0))
