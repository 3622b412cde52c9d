"""Launches whose last rows go to tiles of half the height: row counts on either side of where CUs would end half a tile apart, whole and ragged
lower tiles, columns that are no whole tiles, packed and prepared weights, every kind of output; both experts with routings on either side."""
import pytest
import torch

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
