"""Shift Linears that decode their packed weights on the way into LDS: bit-identical to the same layers on decoded planes, at one,
two, three and many stages of K (odd and even numbers of them), ragged rows and columns, and every epilogue."""
import pytest
import torch

from helpers import dev
from paper_2306_06446_amd import workloads as wl

pytestmark = pytest.mark.gpu


def _case(M, K, N):
    g = torch.Generator(device="cuda")
    g.manual_seed(M + K + N)
    x = torch.randint(-127, 128, (M, K), generator=g, device="cuda", dtype=torch.int8)
    x[-1] = -127
    w = torch.randint(0, 256, (N, K // 2), generator=g, device="cuda", dtype=torch.uint8)
    w[-1] = 0x77                                             # +128 throughout
    return g, x, w


@pytest.mark.parametrize("M,K,N", [
    (1, 64, 4), (64, 128, 64), (65, 192, 100), (197, 1024, 768), (1379, 960, 1028),      # 64 x 64
    (25088, 64, 192), (16385, 128, 256), (12608, 192, 580), (3001, 1088, 1024), (12608, 1536, 384),   # 128 x 64
    (13000, 832, 1000), (16001, 768, 768),                                               # 128 x 64: too little for 192 x 128
    (12609, 768, 772), (12608, 3072, 768), (12000, 832, 1000), (32000, 1280, 320), (11001, 768, 1536),    # 192 x 128
    (40001, 768, 192), (12609, 832, 772), (12608, 2112, 768),                            # 192 x 128: a last column tile half full, odd stages
    (25001, 2048, 512), (50001, 1536, 384),                                              # the planes after all
])
def test_packed_equals_planes(sa, M, K, N):
    g, x, w = _case(M, K, N)
    planes = sa.sa_shift_planes_prepare(w)
    bias = torch.randint(-5000, 5000, (N,), generator=g, device="cuda", dtype=torch.int32)
    ref = sa.sa_shift_linear(x, planes, bias, variant=3)
    assert torch.equal(sa.sa_shift_linear(x, w, bias, variant=1), ref)
    exact = (x[-3:].double() @ torch.from_numpy(_dense(w)).cuda().double().T + bias.double()).to(torch.int32)
    assert torch.equal(ref[-3:], exact)
    res = torch.randn((M, N), generator=g, device="cuda")
    a, = sa.sa_shift_linear_f32(x, w, 0.37, residual=res, variant=1)
    b, = sa.sa_shift_linear_f32(x, planes, 0.37, residual=res, variant=3)
    assert torch.equal(a, b)


@pytest.mark.parametrize("M,K,N", [(65, 192, 101), (16385, 128, 257), (12609, 832, 771)])      # rows of outputs that are no whole 16 bytes
def test_packed_odd_columns(sa, M, K, N):
    _, x, w = _case(M, K, N)
    assert torch.equal(sa.sa_shift_linear(x, w, variant=1), sa.sa_shift_linear(x, sa.sa_shift_planes_prepare(w), variant=3))


# the workspace takes the planes of those layers alone that are decoded before they are multiplied: narrow rows of outputs in pieces
# of lines, padded columns, and what lies beside either
@pytest.mark.parametrize("M,K,N,decoded", [
    (55000, 64, 290, True), (55000, 64, 288, False), (54000, 64, 290, False), (55000, 320, 290, False),
    (60000, 768, 60, True), (60000, 768, 64, False), (60000, 704, 60, False), (40000, 768, 60, False)])
def test_which_layers_are_decoded_first(sa, M, K, N, decoded):
    _, x, w = _case(M, K, N)
    ws = torch.full((2 * N * K,), 77, dtype=torch.uint8, device="cuda")
    got = sa.sa_shift_linear(x, w, variant=1, workspace=ws)
    assert bool((ws != 77).any()) == decoded
    assert torch.equal(got, sa.sa_shift_linear(x, sa.sa_shift_planes_prepare(w), variant=3))


def _dense(w):
    nib = torch.stack([w & 15, w >> 4], dim=-1).flatten(1).cpu().to(torch.int64)
    return (torch.where(nib >= 8, -1, 1) * (1 << (nib & 7))).numpy()


@pytest.mark.parametrize("B,N,H,d", [(1, 50, 2, 64), (5, 300, 6, 128), (32, 197, 12, 64), (50, 500, 4, 64)])
def test_packed_sign_codes(sa, B, N, H, d):
    E = H * d
    _, x, _ = _case(B * N, E, 4)
    w = dev(wl.shift_weights(3, 5, 3 * E, E))
    got = sa.sa_shift_linear_qkv_codes(x, w, B, N, H, 0.5, variant=1)
    ref = sa.sa_shift_linear_qkv_codes(x, sa.sa_shift_planes_prepare(w), B, N, H, 0.5, variant=3)
    assert all(torch.equal(a, b) for a, b in zip(got, ref))


@pytest.mark.parametrize("T,E,hid", [(3000, 384, 1536), (12608, 320, 640)])
def test_packed_mlp(sa, T, E, hid):
    g, x, w1 = _case(T, E, hid)
    w2 = torch.randint(0, 256, (E, hid // 2), generator=g, device="cuda", dtype=torch.uint8)
    lut = dev(wl.activation_lut())
    got = sa.sa_shift_mlp(x, w1, w2, 1e-3, lut, variant=1)
    assert torch.equal(got, sa.sa_shift_mlp(x, sa.sa_shift_planes_prepare(w1), sa.sa_shift_planes_prepare(w2), 1e-3, lut, variant=3))
    for stages in ((1, 2),):                                 # apart, both outputs of the second
        ws = torch.empty(T * hid + 4 * E * hid + 4096, dtype=torch.uint8, device="cuda")
        y = torch.empty((T, E), device="cuda")
        for s in stages:
            y2 = sa.sa_shift_mlp(x, w1, w2, 1e-3, lut, variant=1, stages=s, workspace=ws, y=y, out_scale=0.5)
        assert torch.equal(y2, got) and torch.equal(y, got.float() * 0.5)
