"""The distances that the pipelined Hamming kernel takes from the matrix cores as addresses of its table: every remainder of the 32
keys of a tile and the 16 of a step, the smallest and the largest distance, bit for bit as from popcounts."""
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nbits,dv", [(64, 32), (64, 64), (128, 32), (128, 64), (256, 32), (256, 64)])
@pytest.mark.parametrize("Nk", [1, 15, 16, 17, 31, 32, 33, 47, 48, 49, 127, 128, 129, 144, 161])
def test_distances_of_every_remainder(sa, Nk, nbits, dv):
    g = torch.Generator(device="cuda")
    g.manual_seed(Nk + nbits + dv)
    B, H, Nq, W = 2, 3, 70, nbits // 64
    k = torch.randint(-2 ** 62, 2 ** 62, (B, H, Nk, W), generator=g, device="cuda") * 2 + torch.randint(0, 2, (B, H, Nk, W), generator=g, device="cuda")
    q = torch.randint(-2 ** 62, 2 ** 62, (B, H, Nq, W), generator=g, device="cuda") * 2 + torch.randint(0, 2, (B, H, Nq, W), generator=g, device="cuda")
    at = torch.randint(0, Nk, (B, H, Nq, 1), generator=g, device="cuda").expand(-1, -1, -1, W)
    q[:, :, ::3] = k.gather(2, at)[:, :, ::3]                # distance 0
    q[:, :, 1::3] = ~k.gather(2, at)[:, :, 1::3]             # and nbits
    v = torch.randn((B, Nk, H, dv), generator=g, device="cuda")
    got = sa.sa_hamming_attention_fused(q, k, v, 0.125, nbits, 20.0, variant=2)
    ref = sa.sa_hamming_attention_fused(q, k, v, 0.125, nbits, 20.0, variant=0)
    for a, b in zip(got, ref):
        assert torch.equal(a, b)
    # and the definition: softmax of the similarities, in 64 bits
    bit = torch.arange(64, device="cuda")
    s = [(((t[..., None] >> bit) & 1) * 2 - 1).flatten(-2).double() for t in (q, k)]
    p = torch.softmax(0.125 * (s[0] @ s[1].transpose(-1, -2).contiguous()), -1)
    o = (p @ v.double().transpose(1, 2).contiguous()).transpose(1, 2)
    assert float((got[0].double() - o).abs().max()) <= 1e-4 * float(o.abs().max())


# Units of four tiles: the fewest queries that are split, last units of one row and of whole tiles, one unit for every CU and a few more.
@pytest.mark.parametrize("B,H,Nq,Nk,nbits,dv", [(1, 1, 128, 40, 64, 64), (1, 1, 129, 197, 64, 64), (3, 4, 197, 197, 128, 64), (1, 3, 256, 300, 256, 32),
                                                (2, 2, 385, 129, 64, 32), (64, 2, 133, 17, 128, 32), (43, 3, 133, 17, 128, 32)])
def test_units_of_four_tiles(sa, B, H, Nq, Nk, nbits, dv):
    g = torch.Generator(device="cuda")
    g.manual_seed(Nq + nbits)
    q, k = (torch.randint(-2 ** 62, 2 ** 62, (B, H, n, nbits // 64), generator=g, device="cuda") for n in (Nq, Nk))
    v = torch.randn((B, Nk, H, dv), generator=g, device="cuda")
    got = sa.sa_hamming_attention_fused(q, k, v, 0.125, nbits, 20.0, variant=2)
    ref = sa.sa_hamming_attention_fused(q, k, v, 0.125, nbits, 20.0, variant=0)
    for a, b in zip(got, ref):
        assert torch.equal(a, b)


# Many units of few keys: up to one product's keys they are not pipelined.  Either side of the keys and of the units from which that holds.
@pytest.mark.parametrize("B,H,Nq,Nk,nbits,dv", [(73, 7, 16, 16, 64, 64), (128, 4, 16, 16, 64, 64), (128, 8, 33, 32, 128, 64), (128, 8, 70, 33, 64, 64),
                                                (512, 8, 31, 17, 128, 32), (1365, 3, 32, 1, 64, 32), (64, 16, 300, 9, 64, 64)])
def test_many_units_of_few_keys(sa, B, H, Nq, Nk, nbits, dv):
    test_units_of_four_tiles(sa, B, H, Nq, Nk, nbits, dv)
