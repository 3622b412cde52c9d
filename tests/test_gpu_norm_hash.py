"""A layer whose Q, K, V projection normalises its rows and hashes Q and K itself, against one whose LayerNorm, projection and hash are
launches of their own (the other variants of the Shift Linears): the same integer sums, and bits that the hash's defining chain settles."""
import pytest
import torch

pytestmark = pytest.mark.gpu


def codes_of_the_entry_points(sa, x, gamma1, beta1, wqkv, qkv_scale, proj, B, N, H, nbits):
    """Q's and K's code words as the stages make them one by one, the hash by its defining chain."""
    z = sa.sa_layernorm_quant(x, gamma1, beta1, 1e-6, 32.0, want_ln=False, want_q=True)[1]
    q, k, _ = sa.sa_shift_linear_f32(z, wqkv, qkv_scale, parts=3, variant=0)
    return [sa.sa_binarize(t.view(B, N, H, x.shape[1] // H), proj, nbits, variant=0) for t in (q, k)]


def assert_code_words(layer, codes, T, E):
    """In a layer's workspace they lie behind its int8 rows and Q, K and V."""
    nbytes, up = codes[0].numel() * 8, lambda n: (n + 255) // 256 * 256
    at = up(T * E) + 3 * up(4 * T * E)
    for i, ref in enumerate(codes):
        assert torch.equal(layer.ws[at + i * up(nbytes):][:nbytes].view(torch.int64), ref.flatten()), "QK"[i]


# every width, head width and number of bits; rows that fill no workgroup, one, and more than a round of them; either side of where the
# launch takes over.  qkv_scale brings rows in and out of the range that splits into fp16 terms as it is.
@pytest.mark.parametrize("B,N,H,E,nbits,attention,qkv_scale", [
    (1, 1, 2, 64, 64, 0, 2.0**-12), (3, 77, 1, 64, 64, 0, 2.0**-40), (1, 65, 1, 64, 128, 1, 2.0**30), (2, 131, 1, 64, 256, 0, 2.0**-12),
    (5, 6661, 2, 64, 64, 0, 2.0**-12), (7, 2477, 1, 64, 256, 0, 2.0**-12), (3, 97, 2, 64, 64, 1, 2.0**-140),
    (2, 768, 4, 128, 64, 0, 2.0**-12), (1, 1537, 2, 128, 64, 0, 2.0**20), (16, 191, 2, 128, 128, 1, 2.0**-12), (2, 1536, 2, 128, 128, 0, 2.0**-30),
    (1, 12287, 2, 128, 256, 0, 2.0**-12), (1, 12288, 2, 128, 256, 0, 2.0**-12), (3, 32777, 4, 128, 64, 0, 2.0**-12),
    (3, 32767, 2, 128, 64, 0, 2.0**-12), (2, 5200, 6, 192, 64, 0, 2.0**-12), (54, 199, 3, 192, 64, 1, 2.0**-12),
    (1, 10369, 3, 192, 128, 0, 2.0**-12), (3, 4098, 3, 192, 256, 0, 2.0**-12), (2, 32801, 3, 192, 64, 0, 2.0**-12),
    (1, 13825, 8, 256, 64, 0, 2.0**-12), (128, 127, 4, 256, 64, 1, 2.0**-12), (2, 7001, 4, 256, 128, 0, 2.0**-12),
    (1, 16384, 4, 256, 256, 0, 2.0**-12), (1, 16385, 4, 256, 256, 0, 2.0**-12),
    # a workgroup per chunk: one row, and the last rows that take it, with one more each
    (1, 1, 3, 192, 64, 0, 2.0**-12), (1, 3, 4, 256, 256, 1, 2.0**-12), (1, 1, 4, 128, 64, 0, 2.0**20), (9, 21, 3, 192, 256, 1, 2.0**-30),
    (1, 5440, 1, 64, 128, 0, 2.0**-12), (1, 5441, 1, 64, 128, 0, 2.0**-12), (1, 10880, 2, 64, 64, 0, 2.0**-12), (1, 10881, 1, 64, 64, 0, 2.0**-12),
    (1, 6784, 4, 128, 64, 0, 2.0**-12), (1, 6785, 4, 128, 64, 0, 2.0**-12), (1, 5760, 2, 128, 128, 0, 2.0**-12), (1, 5761, 2, 128, 64, 0, 2.0**-12),
    (1, 3584, 2, 128, 256, 0, 2.0**-12), (1, 3585, 2, 128, 256, 0, 2.0**-12), (8, 224, 3, 192, 64, 1, 2.0**-12), (1, 1793, 6, 192, 64, 0, 2.0**-12),
    (1, 1344, 8, 256, 64, 0, 2.0**-40), (1, 1345, 4, 256, 128, 0, 2.0**-12), (1, 1664, 4, 256, 256, 0, 2.0**-12),
    # the hash in the projection's tiles: rows too wide for a workgroup, and more narrower ones; both tiles, one row more than whole ones of
    # them, columns of V that fill no tile, either side of the fewest rows and of a round of the smaller tiles
    (1, 299, 12, 768, 64, 0, 2.0**-12), (4, 75, 12, 768, 64, 0, 2.0**-40), (1, 700, 6, 384, 128, 1, 2.0**20), (1, 1300, 5, 320, 256, 0, 2.0**-12),
    (5, 197, 6, 384, 64, 0, 2.0**-12), (3, 401, 6, 384, 128, 1, 2.0**-12), (7, 197, 12, 768, 128, 1, 2.0**-140),
    (3, 1792, 12, 768, 256, 0, 2.0**-12), (1, 5377, 12, 768, 64, 0, 2.0**-30), (33, 257, 12, 768, 128, 1, 2.0**-12), (2, 6001, 6, 384, 256, 0, 2.0**20),
    (1, 8000, 5, 320, 128, 0, 2.0**-30), (3, 1111, 7, 448, 64, 0, 2.0**-12), (3, 1111, 14, 448, 64, 1, 2.0**-40), (1, 3000, 12, 384, 64, 0, 2.0**30),
    (7, 450, 6, 192, 64, 0, 2.0**-12), (2, 1600, 3, 192, 128, 1, 2.0**-12), (1, 2600, 4, 256, 256, 0, 2.0**-12), (5, 4001, 8, 256, 64, 0, 2.0**-12),
    (1, 20480, 4, 128, 64, 0, 2.0**-12), (1, 20481, 2, 128, 128, 0, 2.0**-12), (5, 8192, 4, 256, 256, 0, 2.0**-12), (3, 18205, 6, 192, 64, 0, 2.0**-12),
    # packed weights: the last rows that keep launches of their own, and one more
    (3, 1365, 12, 768, 64, 0, 2.0**-12), (1, 4096, 12, 768, 64, 0, 2.0**-12), (8, 1024, 6, 384, 128, 1, 2.0**20), (1, 8193, 6, 384, 256, 0, 2.0**-12),
    (1, 49152, 2, 64, 64, 0, 2.0**-12), (3, 4097, 4, 256, 256, 0, 2.0**-40),
    # either side of where a tile's hash costs more than its launch saves: few rows, a last round of few tiles, prepared and packed weights
    (1, 639, 12, 384, 64, 0, 2.0**-12), (1, 640, 12, 384, 64, 0, 2.0**-12), (4, 192, 12, 768, 64, 0, 2.0**-12), (1, 769, 12, 768, 128, 0, 2.0**-12),
    (1, 1899, 6, 384, 256, 0, 2.0**-12), (1, 1900, 6, 384, 256, 0, 2.0**-140), (2, 4672, 6, 384, 256, 0, 2.0**-12), (1, 9345, 6, 384, 256, 0, 2.0**-12),
    (1, 5376, 4, 256, 256, 0, 2.0**-12), (1, 5377, 4, 256, 256, 0, 2.0**-12), (1, 7808, 5, 320, 256, 0, 2.0**-12), (1, 7809, 5, 320, 256, 0, 2.0**-12),
    (1, 16384, 5, 320, 256, 0, 2.0**-12), (1, 15361, 5, 320, 128, 0, 2.0**-12), (2, 7680, 5, 320, 128, 0, 2.0**-12), (1, 24833, 6, 384, 256, 0, 2.0**-12),
    (1, 65536, 1, 64, 64, 0, 2.0**-12), (1, 65537, 1, 64, 64, 0, 2.0**-12), (1, 90112, 4, 256, 256, 0, 2.0**-12),
])
def test_codes_of_a_layer_hashed_in_the_projection(sa, B, N, H, E, nbits, attention, qkv_scale):
    g = torch.Generator(device="cuda")
    g.manual_seed(N + E + nbits)
    T, hid = B * N, 256
    x = torch.randn((T, E), generator=g, device="cuda")
    x[T // 2] = 0.5                                          # no variance
    if T > 64:
        x[T // 3, 0], x[T // 5, 1] = float("nan"), float("inf")
    gamma1, beta1, gamma2, beta2 = (torch.randn(E, generator=g, device="cuda") for _ in range(4))
    beta1[E // 2:] = 0.0
    w = [torch.randint(0, 256, s, generator=g, device="cuda", dtype=torch.uint8)
         for s in ((3 * E, E // 2), (E, E // 2), (hid, E // 2), (E, hid // 2))]
    w[0][2 * E:] = w[0][2 * E:] & 0x33                       # V small enough for sums of every scale to mean something
    proj = torch.randn((E // H, nbits), generator=g, device="cuda")
    proj[:, 5] = 0.0                                         # columns left to the chain altogether
    proj[:, 11] *= 1e-30
    proj[1:, 17] = 0.0
    lut = torch.arange(-128, 128, device="cuda").clamp(min=0).to(torch.int8)
    codes = codes_of_the_entry_points(sa, x, gamma1, beta1, w[0], qkv_scale, proj, B, N, H, nbits)
    y = []
    for variant in (0, 2, 3):
        if variant == 3:
            w = [sa.sa_shift_planes_prepare(t) for t in w]
        layer = sa.binding.Layer(B=B, N=N, H=H, nbits=nbits, E=E, hid=hid, attention=attention, moe=0, shift_variant=variant, eps=1e-6,
                                 ln_inv_scale=32.0, qkv_scale=qkv_scale, attn_scale=(64.0 * N) ** -0.5, act_inv_scale=32.0 * 2.0**-12 / qkv_scale,
                                 o_scale=2.0**-12, requant_scale=2.0**-11, out_scale=2.0**-12, x=x, gamma1=gamma1, beta1=beta1,
                                 gamma2=gamma2, beta2=beta2, wqkv=w[0], wo=w[1], proj=proj, w1=w[2], w2=w[3], lut=lut)
        y.append(layer.forward().clone())
        assert_code_words(layer, codes, T, E)
    rows = torch.isfinite(x).all(dim=1)
    assert float((y[0] - x)[rows].abs().max()) > 0.0
    for other in y[1:]:
        assert torch.equal(y[0].nan_to_num(nan=3.0), other.nan_to_num(nan=3.0))


# Rows of zeros and columns of zeros, whose bits need no chain, beside a column that is not finite, overflows when squared or is denormal: there
# they do.  Every kernel that hashes in the projection: a workgroup per chunk, all chunks, and the projection's tiles of either height.
@pytest.mark.parametrize("odd", [0.0, float("nan"), float("inf"), 1e30, 1e-40])
@pytest.mark.parametrize("B,N,H,E,nbits", [(1, 130, 3, 192, 64), (2, 300, 4, 256, 256), (3, 4567, 2, 64, 64), (1, 4200, 2, 128, 128),
                                           (1, 16384, 4, 256, 256), (1, 900, 6, 384, 128), (1, 700, 12, 384, 64), (2, 2001, 6, 384, 256),
                                           (2, 6001, 6, 384, 256)])
def test_rows_and_columns_of_zeros(sa, B, N, H, E, nbits, odd):
    g = torch.Generator(device="cuda")
    g.manual_seed(N + E + nbits)
    T, hid = B * N, 256
    x = torch.randn((T, E), generator=g, device="cuda")
    x[torch.rand(T, generator=g, device="cuda") < 0.4] = 0.0
    x[T // 2:T // 2 + 20] = 0.0
    x[T // 3, 0], x[T // 5, 1] = float("nan"), float("inf")
    gamma, beta = torch.randn(E, generator=g, device="cuda"), torch.zeros(E, device="cuda")
    w = [torch.randint(0, 256, s, generator=g, device="cuda", dtype=torch.uint8) for s in ((3 * E, E // 2), (E, E // 2), (hid, E // 2), (E, hid // 2))]
    proj = torch.randn((E // H, nbits), generator=g, device="cuda")
    proj[:, 7], proj[:, 40] = 0.0, -0.0
    proj[3, 21] = odd
    codes = codes_of_the_entry_points(sa, x, gamma, beta, w[0], 2.0**-12, proj, B, N, H, nbits)
    w = [sa.sa_shift_planes_prepare(t) for t in w]
    layer = sa.binding.Layer(B=B, N=N, H=H, nbits=nbits, E=E, hid=hid, attention=0, moe=0, shift_variant=3, eps=1e-6, ln_inv_scale=32.0,
                             qkv_scale=2.0**-12, attn_scale=1.0, act_inv_scale=1.0, o_scale=2.0**-12, requant_scale=2.0**-11, out_scale=2.0**-12, x=x,
                             gamma1=gamma, beta1=beta, gamma2=gamma, beta2=beta, wqkv=w[0], wo=w[1], proj=proj, w1=w[2], w2=w[3],
                             lut=torch.zeros(256, dtype=torch.int8, device="cuda"))
    layer.forward()
    assert_code_words(layer, codes, T, E)
