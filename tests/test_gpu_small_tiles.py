"""Either side of the line between 32 x 32 and 32 x 64 tiles of the matrix-core GEMMs with whole-line stages: one row, ragged rows and
columns, the shortest rows, both experts in one launch."""
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M,K,N", [
    (1, 512, 4), (33, 640, 36), (31, 3072, 100), (192, 512, 1024), (193, 896, 860),         # 32 x 32
    (193, 512, 900), (257, 768, 700), (300, 3072, 1000), (1001, 640, 256),                  # 32 x 64
])
def test_shift_linear(sa, M, K, N):
    g = torch.Generator(device="cuda")
    g.manual_seed(M * K + N)
    x = torch.randint(-127, 128, (M, K), generator=g, device="cuda", dtype=torch.int8)
    w4 = torch.randint(0, 256, (N, K // 2), generator=g, device="cuda", dtype=torch.uint8)
    nib = torch.stack([w4 & 15, w4 >> 4], dim=-1).reshape(N, K).double()
    w = torch.where(nib >= 8, -1.0, 1.0) * torch.exp2(nib % 8)
    ref = (x.double() @ w.T).to(torch.int32)                             # exact: below 2^53
    assert torch.equal(sa.sa_shift_linear(x, sa.sa_shift_planes_prepare(w4), variant=3), ref)


@pytest.mark.parametrize("share", [0.0, 0.5, 1.0])
@pytest.mark.parametrize("T,K,N", [(1, 512, 32), (197, 768, 860), (33, 1024, 100), (300, 512, 700), (1000, 640, 256)])
def test_both_experts(sa, T, K, N, share):
    g = torch.Generator(device="cuda")
    g.manual_seed(T + K + N)
    x = torch.randn((T, K), generator=g, device="cuda")
    xq, xh = sa.sa_quantize_act_half(x, 127.0 / 4.0)
    w4 = torch.randint(0, 256, (N, K // 2), generator=g, device="cuda", dtype=torch.uint8)
    wh = (torch.randn((N, K), generator=g, device="cuda") / K**0.5).half()
    shift = torch.rand(T, generator=g, device="cuda") < share
    logits = torch.stack((torch.where(shift, -1.0, 1.0), torch.where(shift, 1.0, -1.0)), dim=1).contiguous()
    got = sa.sa_moe_linear(xq, xh, logits, w4, wh, 0.01)
    gate = torch.softmax(logits, dim=1).amax(dim=1, keepdim=True)
    ref = sa.sa_moe_linear(xq, xh, logits, w4, wh, 0.01, variant=0)      # a launch for each expert
    assert torch.equal(got[shift], ref[shift])
    # fp32 sums of K exact products of fp16 numbers, |x| . |w| of them in all: K 2^-24 of that, twice for the order, and the gate's
    bound = gate * (xh.float().abs() @ wh.float().abs().T) * (K + 4) * 2.0**-23
    want = gate * (xh.float().double() @ wh.double().T).float()
    assert bool(((got - want).abs() <= bound)[~shift].all())
