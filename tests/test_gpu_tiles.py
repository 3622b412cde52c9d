"""The tiles of the matrix-core GEMMs at the sizes where their choice changes and where a tile can go wrong: one row, one
tile, ragged rows and columns, fewer stages of K than the ring has buffers, rows that end inside a stage."""
import numpy as np
import pytest
import torch

from helpers import dev, host
from paper_2306_06446_amd import workloads as wl

pytestmark = pytest.mark.gpu


def decode(w4):
    nib = np.stack([w4 & 15, w4 >> 4], axis=-1).reshape(w4.shape[0], -1).astype(np.int64)
    return np.where(nib & 8, -1, 1) * (1 << (nib & 7))


@pytest.mark.parametrize("M,K,N", [
    (1, 64, 64), (31, 192, 65), (32, 64, 128), (33, 448, 4),            # 32-row tiles, 64-byte stages
    (1, 512, 64), (65, 640, 132), (197, 3072, 768), (33, 2048, 36),     # 32-row tiles, 128-byte stages
    (4129, 64, 256), (2081, 224, 512), (1300, 96, 1000),                # 64-row tiles, 64-byte stages
    (1379, 512, 900), (965, 3072, 768), (4161, 768, 260),               # 64-row tiles, 128-byte stages
    (6337, 192, 768), (6401, 768, 768), (2003, 96, 1700), (50001, 64, 60),        # 128 x 64, 64-byte stages
    (6400, 3072, 768), (2003, 2048, 1700),                              # 128 x 64, 128-byte stages
    (12609, 160, 1540), (12801, 768, 1300),                             # 128 x 128
    (11521, 192, 1300),                                                 # 256 x 128
    (13001, 2048, 2048),                                                # 192 x 128
])
def test_shift_linear_at_the_borders_of_the_tile_choice(sa, M, K, N):
    w4 = wl.shift_weights(3, 5, N, K)
    g = torch.Generator(device="cuda")
    g.manual_seed(M * K + N)
    x = torch.randint(-127, 128, (M, K), generator=g, device="cuda", dtype=torch.int8)
    x[-1] = 127
    ref = (x.double() @ torch.from_numpy(decode(w4).T.copy()).cuda().double()).to(torch.int32)     # exact: below 2^53
    assert torch.equal(sa.sa_shift_linear(x, dev(w4), variant=1), ref)
    assert torch.equal(sa.sa_shift_linear(x, sa.sa_shift_planes_prepare(dev(w4)), variant=3), ref)


@pytest.mark.parametrize("rows,E,hid", [
    (1, 32, 64), (33, 64, 96), (65, 192, 768), (197, 768, 256),         # 32-row tiles
    (1379, 192, 768), (965, 768, 1024), (1250, 1536, 192),              # 64-row tiles, short and long rows
    (3200, 768, 992), (6500, 128, 512), (3300, 384, 1536),         # fc1: 192 x 128, 128 x 128 with 64-byte stages
    (3300, 512, 1536),                                             # fc2: 128 x 128 with long rows
])
def test_mult_expert_at_the_borders_of_the_tile_choice(sa, rows, E, hid):
    g = torch.Generator(device="cuda")
    g.manual_seed(rows + E + hid)
    x = torch.randn((rows, E), generator=g, device="cuda").half()
    w1 = (torch.randn((hid, E), generator=g, device="cuda") / E ** 0.5).half()
    w2 = (torch.randn((E, hid), generator=g, device="cuda") / hid ** 0.5).half()
    h = torch.nn.functional.gelu(x.float() @ w1.float().T).half()
    ref = h.float() @ w2.float().T
    got = sa.sa_mult_mlp_f16_half(x, w1, w2)
    err = (got - ref).abs()
    assert bool((err <= 1e-3 + 2e-3 * ref.abs()).all()), float(err.max())
    # the same rows picked from a longer list through device-side counts, scattered with a gate
    T = 2 * rows + 3
    xt = torch.randn((T, E), generator=g, device="cuda").half()
    perm = torch.randperm(T, generator=g, device="cuda").to(torch.int32)
    xt[perm[:rows].long()] = x
    counts = torch.tensor([rows, T - rows, 0, 0], dtype=torch.int32, device="cuda")[:2]
    gate = torch.rand(T, generator=g, device="cuda")
    y = torch.full((T, E), 7.0, device="cuda")
    sa.sa_mult_mlp_f16_half(xt, w1, w2, rows=perm, counts=counts, expert=0, max_rows=T, want_out=False, y=y, gate=gate)
    picked = perm[:rows].long()
    err = (y[picked] - gate[picked, None] * ref).abs()
    assert bool((err <= 1e-3 + 2e-3 * ref.abs()).all()), float(err.max())
    rest = perm[rows:].long()
    assert bool((y[rest] == 7.0).all())


@pytest.mark.parametrize("B,N,H,d", [(1, 50, 2, 64), (7, 197, 12, 64), (3, 300, 6, 128), (26, 500, 6, 128), (32, 197, 12, 64),
                                     (1, 40, 8, 64), (4, 200, 4, 64),                     # slices of either stage width
                                     (50, 500, 4, 64), (2, 300, 16, 128), (7, 601, 16, 128)])   # 128 x 128, 128 x 64 and 192 x 128, long rows
def test_sign_codes_of_every_tile_width(sa, B, N, H, d):
    E = H * d
    g = torch.Generator(device="cuda")
    g.manual_seed(B * N)
    x = torch.randint(-127, 128, (B * N, E), generator=g, device="cuda", dtype=torch.int8)
    w = sa.sa_shift_planes_prepare(dev(wl.shift_weights(3, 5, 3 * E, E)))
    qc, kc, v = sa.sa_shift_linear_qkv_codes(x, w, B, N, H, 0.5, variant=3)
    q, k, ref_v = sa.sa_shift_linear_f32(x, w, 0.5, parts=3, variant=3)
    assert torch.equal(v.flatten(), ref_v.flatten())
    weight = torch.tensor([1 << j for j in range(63)] + [-(1 << 63)], device="cuda")
    for got, f in ((qc, q), (kc, k)):
        bits = (f.view(B, N, H, d // 64, 64) >= 0).to(torch.int64)
        assert torch.equal(got, (bits * weight).sum(-1).permute(0, 2, 1, 3))


@pytest.mark.parametrize("rows", [1024, 16384])                          # 32-row tiles, 128 x 128
def test_gelu_of_every_finite_half(sa, rows):
    bits = torch.arange(65536, device="cuda").remainder(65536).to(torch.int32)
    x = torch.where(bits < 32768, bits, bits - 65536).to(torch.int16).view(torch.float16)
    x = torch.where(torch.isfinite(x), x, torch.zeros_like(x)).view(1024, 64).repeat(rows // 1024, 1)
    eye = torch.eye(64, device="cuda").half()
    got = sa.sa_mult_mlp_f16_half(x.contiguous(), eye, eye).double()     # identity weights: the hidden rows as they are
    a = x.double()
    ref = 0.5 * a * torch.special.erfc(-a * 0.5 ** 0.5)
    ulp = torch.exp2(torch.floor(torch.log2(ref.abs().clamp(min=2.0 ** -14))) - 10)
    assert float(((got - ref).abs() / ulp).max()) <= 0.505
