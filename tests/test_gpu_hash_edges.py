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


@pytest.mark.parametrize("N,nbits", [(4096, 128), (4128, 128), (4128, 256)])     # workgroups of 64, 128 and (d = 128 apart) 256 columns
@pytest.mark.parametrize("d", [32, 64, 128])
def test_bits_are_the_chains_at_the_margin(sa, d, N, nbits):
    """Rows whose product with a column is about what the margin allows for, at the lengths between which rows split unscaled; rows
    whose upper and lower fp16 terms pull that product to different sides; columns whose squares underflow."""
    g = torch.Generator(device="cuda")
    g.manual_seed(d)
    H = 2
    proj = torch.randn((d, nbits), generator=g, device="cuda")
    unit = (proj / proj.norm(dim=0)).double()
    col = torch.randint(0, nbits, (1, N, H), generator=g, device="cuda")
    r = unit.t()[col]                                                       # [1, N, H, d]
    limits = torch.tensor([0.25, 0.25 * (1 - 2 ** -12), 0.25 * (1 + 2 ** -12), 0.0625, 0.5, 1.4, 4096.0, 4096.0 * 1.001],
                          device="cuda", dtype=torch.float64)
    length = limits[torch.randint(0, 8, (1, N, H, 1), generator=g, device="cuda")]
    theta = {32: 2.0 ** -16, 64: 2.0 ** -15, 128: 2.0 ** -14}[d]
    x = torch.randn((1, N, H, d), generator=g, device="cuda", dtype=torch.float64)
    x -= (x * r).sum(-1, keepdim=True) * r
    x = x / x.norm(dim=-1, keepdim=True)
    near = theta * (3 * torch.rand((1, N, H, 1), generator=g, device="cuda", dtype=torch.float64) - 1.5)
    q = ((x + near * r) * length).float()
    up = (x * length).half().double()                                       # k: upper terms + lower terms of the opposite side
    lower = -torch.sign((up * r).sum(-1, keepdim=True)) * r.sign() * up.abs() * 2.0 ** -12.2
    k = (up + lower).float()
    slim = proj.clone()
    slim[:, ::3] *= 2.0 ** -75
    slim[:, 1::3] *= 2.0 ** -60
    for p in (proj, slim):
        codes = [torch.zeros((1, H, N, nbits // 64), dtype=torch.int64, device="cuda") for _ in range(2)]
        sa.sa_binarize_pair(q, k, p, nbits, *codes)
        for t, c in zip((q, k), codes):
            assert torch.equal(c, sa.sa_binarize(t, p, nbits, variant=0))


# either side of the 512 tiles of 32 rows (both tensors') up to which a workgroup has fewer columns, and, at 256, of the 192 MiB of rows
# from which they are loaded as a stream
@pytest.mark.parametrize("d,nbits,N", [(d, nbits, N) for d in (32, 64, 128) for nbits in (128, 256) for N in (8187, 8193)] +
                         [(32, 256, 786399), (32, 256, 786401), (64, 256, 393183), (64, 256, 393185)])
def test_either_side_of_the_rules(sa, d, nbits, N):
    test_bits_are_the_chains(sa, 1, N, 1, d, nbits, "plain")


@pytest.mark.parametrize("d,nbits", [(32, 64), (64, 64), (64, 192), (128, 64), (128, 320)])
def test_workgroups_of_64_columns_over_many_tiles(sa, d, nbits):
    """More tiles than wavefronts: two workgroups of four wavefronts to a CU, each with several tiles, the last ones uneven."""
    g = torch.Generator(device="cuda")
    g.manual_seed(d + nbits)
    x = [torch.randn((11, 3333, 2, d), generator=g, device="cuda") for _ in range(2)]       # 73326 rows: 2 x 2292 tiles
    proj = torch.randn((d, nbits), generator=g, device="cuda")
    codes = sa.sa_binarize_pair(x[0], x[1], proj, nbits)
    for t, c in zip(x, codes):
        assert torch.equal(c, sa.sa_binarize(t, proj, nbits, variant=0))


@pytest.mark.parametrize("N", [65504, 65536, 65537, 131073, 200001])
def test_short_tiles_shared_out_one_by_one(sa, N):
    """32 to 64 columns: Q and K are one tile of each wavefront less two, one each, two over, and up to four each."""
    g = torch.Generator(device="cuda")
    g.manual_seed(N)
    x = [torch.randn((1, N, 1, 32), generator=g, device="cuda") for _ in range(2)]
    proj = torch.randn((32, 64), generator=g, device="cuda")
    for t, c in zip(x, sa.sa_binarize_pair(x[0], x[1], proj, 64)):
        assert torch.equal(c, sa.sa_binarize(t, proj, 64, variant=0))


@pytest.mark.parametrize("B,N,d", [(4, 1024, 64), (5, 1000, 64), (33, 500, 32)])
def test_hash_that_routes_along(sa, B, N, d):
    """Around the number of tokens from which the workgroups that also route are larger ones: what the hash leaves is the same (the
    attention output of a block with a router and of one without, bit for bit), and so is the routing."""
    g = torch.Generator(device="cuda")
    g.manual_seed(N)
    H, T, nbits, E, hid = 2, B * N, 64, 2 * d, 128

    def randn(*shape):
        return torch.randn(shape, generator=g, device="cuda")

    kw = dict(B=B, N=N, H=H, d=d, nbits=nbits, dv=d, attention=0, attn_scale=1.0 / (N * nbits) ** 0.5, q=randn(B, N, H, d),
              k=randn(B, N, H, d), v=randn(B, N, H, d), proj=randn(d, nbits))
    plain, _ = sa.binding.Block(hid=0, moe=False, **kw).forward()
    w = [torch.randint(0, 256, s, generator=g, device="cuda", dtype=torch.uint8) for s in ((hid, E // 2), (E, hid // 2))]
    mw = [randn(hid, E).half() * 0.1, randn(E, hid).half() * 0.1]
    lut = torch.arange(-128, 128, device="cuda").to(torch.int8)
    logits = randn(T, 2)
    mlp = dict(w1=w[0], w2=w[1], lut=lut, mw1=mw[0], mw2=mw[1], act_inv_scale=30.0, requant_scale=1e-3, out_scale=1e-3)
    o, y = sa.binding.Block(hid=hid, moe=True, logits=logits, **mlp, **kw).forward()
    assert torch.equal(o, plain)
    # every row of y as its expert alone gives it, times its gate
    expert = (logits[:, 1] > logits[:, 0]).long()
    gate = torch.softmax(logits.double(), 1).gather(1, expert[:, None])
    ys = []
    for e in (0, 1):
        one = torch.full((T, 2), -200.0, device="cuda")
        one[:, e] = 0.0                                    # gate 1
        ys.append(sa.binding.Block(hid=hid, moe=True, logits=one, **mlp, **kw).forward()[1].double())
    ref = torch.where(expert[:, None] == 0, ys[0], ys[1]) * gate
    assert bool(((y.double() - ref).abs() <= 1e-5 * ref.abs() + 1e-6 * float(ref.square().mean().sqrt())).all())
