"""Launches whose last rows go to tiles of half the height: row counts on either side of where CUs would end half a tile apart, whole and ragged
lower tiles, columns that are no whole tiles, packed and prepared weights, int32, fp32, sign-code, int8 table and scattered outputs; both experts
with routings on either side, as Linears and as the first layer of a block."""
import pytest
import torch

from test_gpu_hidden_columns import test_block_against_separate_launches as block_against_separate_launches

pytestmark = pytest.mark.gpu


def weights(g, N, K):
    w4 = torch.randint(0, 256, (N, K // 2), generator=g, device="cuda", dtype=torch.uint8)
    nib = torch.stack([w4 & 15, w4 >> 4], dim=-1).reshape(N, K).double()
    return w4, torch.where(nib >= 8, -1.0, 1.0) * torch.exp2(nib % 8)


# tiles of 128 x 64, 8 XCDs, 32 CUs each: one to 16 tiles more than whole rounds of CUs take the lower ones, 17 do not, nor does a second round
@pytest.mark.parametrize("M,K,N", [
    (12608, 1536, 384), (11300, 384, 384), (11233, 384, 384), (13313, 384, 384), (13824, 128, 384), (13825, 128, 384),
    (20033, 512, 256), (25089, 1024, 192), (9001, 1024, 500), (10240, 320, 320), (16500, 64, 320),
])
def test_shift_linear(sa, M, K, N):
    g = torch.Generator(device="cuda")
    g.manual_seed(M + K + N)
    x = torch.randint(-127, 128, (M, K), generator=g, device="cuda", dtype=torch.int8)
    w4, w = weights(g, N, K)
    ref = (x.double() @ w.T).to(torch.int32)                             # exact: below 2^53
    planes = sa.sa_shift_planes_prepare(w4)
    assert torch.equal(sa.sa_shift_linear(x, w4), ref)
    assert torch.equal(sa.sa_shift_linear(x, planes, variant=3), ref)
    residual = torch.randn((M, N), generator=g, device="cuda")
    y = sa.sa_shift_linear_f32(x, planes, 0.5, residual=residual, variant=3)[0]
    want = ref.float().double() * 0.5 + residual.double()                # one fma: one rounding of the exact value
    assert torch.equal(y, want.float())


def test_sign_codes(sa):
    B, N, H, E = 4, 3152, 2, 128
    g = torch.Generator(device="cuda")
    g.manual_seed(1)
    x = torch.randint(-127, 128, (B * N, E), generator=g, device="cuda", dtype=torch.int8)
    w4, w = weights(g, 3 * E, E)
    acc = x.double() @ w.T
    qc, kc, v = sa.sa_shift_linear_qkv_codes(x, sa.sa_shift_planes_prepare(w4), B, N, H, 0.25, variant=3)
    assert torch.equal(v, (acc[:, 2 * E:] * 0.25).float())
    bits = torch.arange(64, device="cuda")
    for i, c in enumerate((qc, kc)):
        want = (acc[:, i * E:(i + 1) * E] >= 0).view(B, N, H, 64).permute(0, 2, 1, 3)
        assert torch.equal(((c >> bits) & 1).bool(), want)


@pytest.mark.parametrize("T,K,N,share", [(12608, 768, 768, 0.70), (12608, 768, 768, 0.40), (11000, 768, 768, 0.5), (11001, 768, 768, 1.0),
                                         (7003, 512, 1100, 0.5), (25088, 384, 384, 0.61), (12608, 768, 768, 0.0)])
def test_both_experts(sa, T, K, N, share):
    g = torch.Generator(device="cuda")
    g.manual_seed(T + K + int(100 * share))
    x = torch.randn((T, K), generator=g, device="cuda")
    xq, xh = sa.sa_quantize_act_half(x, 127.0 / 4.0)
    w4, _ = weights(g, N, K)
    wh = (torch.randn((N, K), generator=g, device="cuda") / K**0.5).half()
    shift = torch.rand(T, generator=g, device="cuda") < share
    logits = torch.stack((torch.where(shift, -1.0, 1.0), torch.where(shift, 1.0, -1.0)), dim=1).contiguous()
    y = torch.full((T, N), float("nan"), device="cuda")
    got = sa.sa_moe_linear(xq, xh, logits, w4, wh, 0.01, y=y)
    ref = sa.sa_moe_linear(xq, xh, logits, w4, wh, 0.01, variant=0)      # a launch for each expert
    assert torch.equal(got[shift], ref[shift])
    # fp32 sums of K products in two orders, as test_gpu_split_tiles.py allows
    torch.testing.assert_close(got[~shift], ref[~shift], rtol=1e-4, atol=1e-4)


# first layers (int8 through the table) and second ones (scattered fp32 rows) of which either has lower tiles; rows as they are and picked
@pytest.mark.parametrize("M,E,hid", [(6000, 320, 768), (7001, 320, 768), (12608, 384, 1536), (6499, 320, 768)])
@pytest.mark.parametrize("picked", [False, True])
def test_shift_mlp(sa, M, E, hid, picked):
    g = torch.Generator(device="cuda")
    g.manual_seed(M + E)
    T = M + 50
    x = torch.randint(-127, 128, (T, E), generator=g, device="cuda", dtype=torch.int8)
    (w1, f1), (w2, f2) = weights(g, hid, E), weights(g, E, hid)
    lut = torch.randint(-128, 128, (256,), generator=g, device="cuda", dtype=torch.int8)
    rows = torch.randperm(T, generator=g, device="cuda")[:M].to(torch.int32) if picked else torch.arange(M, device="cuda", dtype=torch.int32)
    rq = 2.0**-11                                                        # a power of two: one rounding, of the product, to even
    h = lut[(x[rows.long()].double() @ f1.T * rq).round().clamp(-127, 127).long() + 128]
    want = torch.full((T, E), 7.0, device="cuda")
    want[rows.long()] = (h.double() @ f2.T).float() * 0.5
    planes = sa.sa_shift_planes_prepare(w1), sa.sa_shift_planes_prepare(w2)
    for w, variant in (((w1, w2), 1), (planes, 3)):
        y = torch.full((T, E), 7.0, device="cuda")
        sa.sa_shift_mlp(x, *w, rq, lut, want_y2=False, y=y, out_scale=0.5, variant=variant, rows=rows, max_rows=M)
        assert torch.equal(y, want)


@pytest.mark.parametrize("share", [0.0, 0.15, 0.4, 0.65, 0.9, 1.0])
@pytest.mark.parametrize("B,N,H,hid", [(1, 5617, 6, 1536), (1, 8501, 4, 1024)])
def test_block_of_both_experts(sa, B, N, H, hid, share):
    block_against_separate_launches(sa, B, N, H, hid, share)
