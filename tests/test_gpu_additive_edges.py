"""The matrix-core Add kernels where their splitting of the work changes or can go wrong: fewer tokens than one step, ragged
steps, code words that do not pair up, many short sequences, partials summed by Q(K^T V) or by a kernel of their own."""
import pytest
import torch

pytestmark = pytest.mark.gpu


def codes(g, *shape):
    return torch.randint(-2**63, 2**63 - 1, shape, generator=g, device="cuda", dtype=torch.int64)


def bits_of(c):
    """int64 code words [..., W] -> float64 {0, 1} [..., 64 W]."""
    j = torch.arange(64, device=c.device)
    return ((c.unsqueeze(-1) >> j) & 1).flatten(-2).double()


@pytest.mark.parametrize("B,H,Nq,Nk,W,dv", [
    (1, 1, 1, 1, 1, 32), (1, 2, 33, 15, 1, 64), (2, 1, 31, 17, 2, 32), (1, 3, 64, 129, 2, 64),      # below and around one step
    (1, 2, 40, 300, 3, 64), (1, 1, 20, 500, 5, 32), (1, 2, 70, 257, 6, 128),                        # words that do not pair up
    (2, 2, 300, 4097, 4, 64), (1, 1, 513, 9000, 4, 128), (3, 1, 95, 2000, 4, 32),                   # many partials
    (40, 13, 50, 49, 1, 32), (30, 18, 37, 197, 2, 64), (44, 12, 33, 20, 1, 64),                     # many short sequences
    (1, 3, 197, 197, 1, 64), (2, 2, 256, 255, 2, 128), (43, 6, 512, 512, 1, 64), (22, 12, 300, 511, 2, 32),  # both products in one launch
    (43, 6, 513, 512, 2, 64), (43, 6, 100, 513, 1, 32),                                             # one token too many for that
    (8, 4, 8192, 300, 1, 64),                                                                       # 32-tile passes of Q(K^T V)
])
def test_both_code_modes_against_fp64(sa, B, H, Nq, Nk, W, dv):
    g = torch.Generator(device="cuda")
    g.manual_seed(Nq * Nk + W)
    q, k = codes(g, B, H, Nq, W), codes(g, B, H, Nk, W)
    v = torch.randn((B, Nk, H, dv), generator=g, device="cuda")
    nbits, vt = 64 * W, v.double().permute(0, 2, 1, 3).contiguous()
    kb, qb = bits_of(k), bits_of(q)
    for zero_one in (False, True):
        ks, qs = (kb, qb) if zero_one else (2 * kb - 1, 2 * qb - 1)
        kv_ref = torch.matmul(ks.transpose(-1, -2).contiguous(), vt)
        ref = torch.matmul(qs, kv_ref)
        if zero_one:
            ksum_ref = kb.sum(2)
            ref = ref / (torch.matmul(qb, ksum_ref.unsqueeze(-1)) + 1e-6)
            out, kv, ksum = sa.sa_linear_attention_01(q, k, v, 1e-6, nbits)
            assert torch.equal(ksum.long(), ksum_ref.long())
            parts = sa.sa_linear_attention_01(None, k, v, 1e-6, nbits, phases=1)
            again = sa.sa_linear_attention_01(q, None, None, 1e-6, nbits, phases=2, kv=parts[1], ksum=parts[2])
            assert torch.equal(parts[2], ksum)
        else:
            scale = 1.0 / (Nk * nbits) ** 0.5
            ref = ref * scale
            out, kv = sa.sa_additive_attention(q, k, v, scale, nbits)
            parts = sa.sa_additive_attention(None, k, v, scale, nbits, phases=1)
            again = sa.sa_additive_attention(q, None, None, scale, nbits, phases=2, kv=parts[1])
        assert torch.equal(parts[1], kv) and torch.equal(again[0], out)        # one call or two: the same sums
        ref = ref.permute(0, 2, 1, 3)
        err_kv, err = (kv.double() - kv_ref).abs(), (out.double() - ref).abs()
        assert bool((err_kv <= 1e-4 * kv_ref.abs() + 1e-5 * max(1.0, float(kv_ref.square().mean().sqrt()))).all())
        assert bool((err <= 1e-4 * ref.abs() + 1e-5).all()), float(err.max())


@pytest.mark.parametrize("Nq", [0, 1])                     # K^T V alone, both products in one launch
def test_rows_of_a_ragged_step_more_than_4_gib_apart(sa, Nq):
    B, H, Nk, dv = 1, 600_000, 15, 128                     # 14 rows of V take 14 * H * dv * 4 = 4.30e9 > 2^32 bytes
    g = torch.Generator(device="cuda")
    g.manual_seed(1)
    k = codes(g, B, H, Nk, 1)
    v = torch.randn((B, Nk, H, dv), generator=g, device="cuda")
    if Nq:
        q = codes(g, B, H, Nq, 1)
        out, kv = sa.sa_additive_attention(q, k, v, 0.125, 64)
    else:
        kv = sa.sa_additive_attention(None, k, v, 0.125, 64, phases=1)[1]
    heads = torch.cat((torch.tensor([0, 1, H // 2, H - 2, H - 1], device="cuda"), torch.randint(0, H, (200,), generator=g, device="cuda")))
    ks = 2 * bits_of(k[0, heads]) - 1                      # [heads, Nk, 64]
    ref = torch.matmul(ks.transpose(-1, -2).contiguous(), v[0][:, heads].double().transpose(0, 1).contiguous())
    err = (kv[0, heads].double() - ref).abs()
    assert bool((err <= 1e-4 * ref.abs() + 1e-5 * float(ref.square().mean().sqrt())).all()), float(err.max())
    if Nq:
        o_ref = 0.125 * torch.matmul(2 * bits_of(q[0, heads]) - 1, ref)
        err = (out[0][:, heads].double().transpose(0, 1) - o_ref).abs()
        assert bool((err <= 1e-4 * o_ref.abs() + 1e-5 * float(o_ref.square().mean().sqrt())).all()), float(err.max())


# passes of 16 wavefronts over two tiles each: a whole pass and a ragged tile behind it, every code width
@pytest.mark.parametrize("W", [1, 2, 4])
def test_passes_of_sixteen_wavefronts(sa, W):
    test_both_code_modes_against_fp64(sa, 8, 4, 8200, 40, W, 64)


# K^T V in two, three, five and six partials, summed by Q(K^T V)
@pytest.mark.parametrize("H,N,W,dv", [(12, 137, 4, 64), (8, 300, 4, 32), (3, 1200, 2, 32), (2, 1500, 1, 64)])
def test_a_few_partials(sa, H, N, W, dv):
    test_both_code_modes_against_fp64(sa, 1, H, N, N, W, dv)


# 64 bits: two to sixteen partials, eight of which are in flight together; half of a head's columns to a workgroup; passes of sixteen wavefronts
@pytest.mark.parametrize("H,Nq,Nk,dv", [(1, 40, 500, 32), (1, 257, 1790, 32), (2, 70, 2048, 32), (1, 300, 2300, 32), (3, 33, 4096, 32),
                                        (1, 513, 3900, 32), (2, 600, 2040, 64), (2, 100, 1000, 128), (8, 32777, 1500, 64)])
def test_partials_summed_by_quads(sa, H, Nq, Nk, dv):
    test_both_code_modes_against_fp64(sa, 1, H, Nq, Nk, 1, dv)


# 64 bits in two partials: few workgroups, and more than two for a CU, which sum by quads
@pytest.mark.parametrize("B,H,N,dv", [(1, 12, 400, 64), (43, 3, 300, 64), (50, 4, 400, 64), (1, 127, 512, 128)])
def test_two_partials(sa, B, H, N, dv):
    test_both_code_modes_against_fp64(sa, B, H, N, N, 1, dv)
