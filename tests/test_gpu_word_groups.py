"""K^T V of codes of three words and more, two or four of them to a workgroup: with partials and without, V up to 32 and 64 MiB and beyond them, partials
that Q(K^T V) would sum itself, ragged steps and words that do not pair up, both kinds of codes; and how far two words' sums are from exact ones."""
import pytest
import torch

pytestmark = pytest.mark.gpu


def bits_of(c):
    """int64 code words [..., W] -> float64 {0, 1} [..., 64 W]."""
    j = torch.arange(64, device=c.device)
    return ((c.unsqueeze(-1) >> j) & 1).flatten(-2).double()


@pytest.mark.parametrize("B,H,N,W,dv", [
    (1, 4, 5471, 4, 64), (1, 3, 197, 4, 64), (2, 2, 257, 3, 32), (1, 2, 1027, 5, 64), (1, 1, 3000, 6, 128), (3, 2, 700, 8, 32),      # two words
    (32, 8, 60, 4, 64), (100, 6, 130, 3, 32),                                                       # no partials: four
    (8, 4, 4096, 4, 64), (8, 4, 4097, 4, 64), (16, 12, 1365, 4, 64), (16, 12, 1366, 4, 64),         # V of 32 MiB and a little more, of 64
    (32, 1, 3136, 4, 32), (16, 1, 2049, 4, 64),                                                     # Q(K^T V) would sum the partials of two words
])
@pytest.mark.parametrize("zero_one", [False, True])
def test_against_fp64(sa, B, H, N, W, dv, zero_one):
    g = torch.Generator(device="cuda")
    g.manual_seed(B * N + W)
    k = torch.randint(-2**63, 2**63 - 1, (B, H, N, W), generator=g, device="cuda", dtype=torch.int64)
    v = torch.randn((B, N, H, dv), generator=g, device="cuda")
    bits = bits_of(k)
    if zero_one:
        _, kv, ksum = sa.sa_linear_attention_01(None, k, v, 1e-6, 64 * W, phases=1)
        assert torch.equal(ksum.long(), bits.sum(2).long())
    else:
        kv = sa.sa_additive_attention(None, k, v, 1.0, 64 * W, phases=1)[1]
        bits = 2 * bits - 1
    ref = torch.matmul(bits.transpose(-1, -2).contiguous(), v.double().permute(0, 2, 1, 3).contiguous())
    # sums of exact products in fp32, in parts: N roundings of partial sums of rms up to sqrt(N) would be N 2^-24 of them at worst; their
    # rms is sqrt(N / 16) 2^-25 of the result's, and ten times that covers 10^7 of them
    bound = 10 * (N / 16) ** 0.5 * 2.0**-25 * N**0.5 + 2.0**-22 * N**0.5
    assert float((kv.double() - ref).abs().max()) <= bound


# The relative error of K^T V (2-norm, these inputs) with four words to a workgroup, which two take the place of here: the same fp32 terms in
# twice as many partials, added one after the other.  Two words' sums are in another order and may be no further off; they measured 2 to 9 % less.
@pytest.mark.parametrize("B,H,N,W,dv,four", [
    (1, 4, 16384, 4, 64, 1.249e-7), (1, 4, 5471, 4, 64, 1.079e-7), (2, 4, 8000, 4, 64, 1.184e-7), (4, 4, 8192, 4, 64, 1.372e-7),
    (2, 12, 197, 4, 64, 7.776e-8), (1, 3, 197, 4, 64, 7.773e-8), (1, 4, 9973, 3, 64, 1.218e-7), (1, 2, 6000, 8, 32, 1.143e-7),
])
def test_no_further_off_than_four_words(sa, B, H, N, W, dv, four):
    errors = []
    for seed in range(4):
        g = torch.Generator(device="cuda")
        g.manual_seed(seed)
        k, _ = (torch.randint(-2**63, 2**63 - 1, (B, H, N, W), generator=g, device="cuda", dtype=torch.int64) for _ in range(2))
        v = torch.randn((B, N, H, dv), generator=g, device="cuda")
        kv = sa.sa_additive_attention(None, k, v, 1.0, 64 * W, phases=1)[1]
        ref = torch.stack([(2 * bits_of(k[b, h]) - 1).T.contiguous() @ v[b, :, h].double() for b in range(B) for h in range(H)]).view(kv.shape)
        errors.append(float((kv.double() - ref).norm() / ref.norm()))
    assert sum(errors) / 4 <= four
