"""GPU parity: the HIP library, called through its C ABI, against the CPU oracle.

Integer / bit / index results must be bit-exact; floating-point attention outputs must
meet 1e-4 relative + 1e-5 absolute (fp32 accumulation) on the scaled output.
Sizes here finish in seconds on the oracle and still span several tiles with ragged tails.
"""
import math

import numpy as np
import pytest
import torch

import oracle
from helpers import ATTN_ATOL, ATTN_RTOL, assert_close, codes_host, dev, host, kv_tolerance
from paper_2306_06446_amd import workloads as wl

pytestmark = pytest.mark.gpu


# ------------------------------------------------------------------ binarize ----

@pytest.mark.parametrize("B,N,H,d,nbits", [
    (1, 197, 3, 64, 64),      # c1
    (2, 130, 1, 32, 64),      # c2 widths, ragged
    (2, 197, 12, 64, 128),    # c4 widths
    (1, 300, 4, 64, 256),     # c5 widths
    (1, 1, 1, 128, 192),      # single row, d = 128
    (3, 64, 2, 64, 64),       # exact chunk
])
def test_binarize_projection_bit_exact(sa, B, N, H, d, nbits):
    g = np.random.default_rng([1, B, N, H, d, nbits])
    x = g.standard_normal((B, N, H, d), dtype=np.float32)
    pr = g.standard_normal((d, nbits), dtype=np.float32)
    ref = oracle.binarize(x, pr, nbits)
    for variant in (0, 1, None):      # chain on the VALU, matrix-core pre-pass + exact fallback, default
        got = codes_host(sa.sa_binarize(dev(x), dev(pr), nbits, variant=variant))
        assert got.shape == ref.shape
        assert np.array_equal(got, ref), "variant %s" % variant


@pytest.mark.parametrize("variant", [0, 1])
def test_binarize_degenerate_rows_bit_exact(sa, variant):
    """Data on which the matrix-core pre-pass settles nothing: zero rows, rows orthogonal to many hash
    columns, huge and tiny magnitudes, NaN / Inf.  Every such bit must come from the defining chain."""
    g = np.random.default_rng(8)
    d, nbits = 64, 128
    x = g.standard_normal((1, 300, 2, d), dtype=np.float32)
    pr = g.standard_normal((d, nbits), dtype=np.float32)
    pr[:, 5] = 0.0                      # a dead hash column
    pr[32:, 9] = 0.0
    x[0, 0:40] = 0.0                    # zero rows
    x[0, 40:60, :, 32:] = 0.0
    x[0, 40:60, :, :32] = 1.0
    x[0, 60:70] *= np.float32(1e30)     # squares overflow
    x[0, 70:80] *= np.float32(1e-30)    # squares underflow
    x[0, 80:90] *= np.float32(1e-38)    # denormal products
    x[0, 90, 0, 3] = np.nan
    x[0, 91, 1, 7] = np.inf
    x[0, 92, 0, 0] = -np.inf
    x[0, 100:140] = np.round(x[0, 100:140] * 2) / 2    # many exact ties at zero are likely
    pr_i = np.round(pr * 2) / 2
    for p in (pr, pr_i.astype(np.float32)):
        ref = oracle.binarize(x, p, nbits)
        got = codes_host(sa.sa_binarize(dev(x), dev(p), nbits, variant=variant))
        assert np.array_equal(got, ref)


@pytest.mark.parametrize("variant", [0, 1])
def test_binarize_near_cancelling_rows_bit_exact(sa, variant):
    """Rows built to make many projections cancel almost exactly: only the defined
    summation order reproduces these signs."""
    g = np.random.default_rng(2)
    d, nbits = 64, 128
    x = g.standard_normal((1, 257, 2, d), dtype=np.float32)
    pr = g.standard_normal((d, nbits), dtype=np.float32)
    x64 = x.astype(np.float64)
    # last coordinate chosen so that bit (row % nbits) has a projection near zero
    for n in range(x.shape[1]):
        for h in range(2):
            j = (n * 2 + h) % nbits
            s = x64[0, n, h, : d - 1] @ pr[: d - 1, j].astype(np.float64)
            x[0, n, h, d - 1] = np.float32(-s / np.float64(pr[d - 1, j]))
    ref = oracle.binarize(x, pr, nbits)
    got = codes_host(sa.sa_binarize(dev(x), dev(pr), nbits, variant=variant))
    assert np.array_equal(got, ref)


def test_binarize_sign_mode_bit_exact(sa):
    g = np.random.default_rng(3)
    x = g.standard_normal((2, 77, 3, 128), dtype=np.float32)
    x[0, 0, 0, :8] = [0.0, -0.0, np.nan, np.inf, -np.inf, 1e-45, -1e-45, 1.0]
    ref = oracle.binarize(x, None, 128)
    got = codes_host(sa.sa_binarize(dev(x), None, 128))
    assert np.array_equal(got, ref)


@pytest.mark.parametrize("B,N,H,d,nbits", [(2, 197, 12, 64, 128), (1, 300, 4, 64, 256), (2, 130, 1, 32, 64)])
def test_binarize_pair_bit_exact(sa, B, N, H, d, nbits):
    """Two tensors in one launch."""
    g = np.random.default_rng([12, B, N, H, d, nbits])
    q = g.standard_normal((B, N, H, d), dtype=np.float32)
    k = g.standard_normal((B, N, H, d), dtype=np.float32)
    k[0, 0, 0, :] = 0.0                                     # a parked row in the second tensor
    pr = g.standard_normal((d, nbits), dtype=np.float32)
    qc, kc = sa.sa_binarize_pair(dev(q), dev(k), dev(pr), nbits)
    assert np.array_equal(codes_host(qc), oracle.binarize(q, pr, nbits))
    assert np.array_equal(codes_host(kc), oracle.binarize(k, pr, nbits))


def test_binarize_pair_without_projection_is_two_sign_hashes(sa):
    g = np.random.default_rng(13)
    q = g.standard_normal((2, 70, 3, 64), dtype=np.float32)
    k = g.standard_normal((2, 70, 3, 64), dtype=np.float32)
    qc, kc = sa.sa_binarize_pair(dev(q), dev(k), None, 64)
    assert np.array_equal(codes_host(qc), oracle.binarize(q, None, 64))
    assert np.array_equal(codes_host(kc), oracle.binarize(k, None, 64))


# -------------------------------------------------------- additive attention ----

@pytest.mark.parametrize("valu", [0, 4], ids=["mfma", "valu"])
@pytest.mark.parametrize("B,H,Nq,Nk,nbits,dv", [
    (1, 3, 197, 197, 64, 64),     # c1
    (2, 1, 777, 777, 64, 32),     # c2 widths
    (1, 2, 1500, 1500, 256, 64),  # c5 widths, several splits
    (2, 2, 65, 300, 128, 128),    # Nq != Nk, dv = 128
    (1, 1, 1, 1, 64, 32),         # degenerate
    (1, 2, 130, 257, 192, 32),    # three code words: K^T V on the matrix cores, Q(K^T V) on the vector ALU
    (1, 1, 40, 500, 384, 64),     # six code words: two word groups, the second half empty
    (1, 1, 90, 129, 256, 128),    # K^T V planes too large for the LDS: Q(K^T V) on the vector ALU
])
def test_additive_attention_matches_oracle(sa, B, H, Nq, Nk, nbits, dv, valu):
    q = wl.random_codes(1, (B, H, Nq), nbits)
    k = wl.random_codes(2, (B, H, Nk), nbits)
    v = np.random.default_rng([4, B, H, Nk, dv]).standard_normal((B, Nk, H, dv), dtype=np.float32)
    scale = float(np.float32(1.0 / math.sqrt(Nk * nbits)))
    o_ref, kv_ref = oracle.additive_attention(q, k, v, nbits, scale)
    out, kv = sa.sa_additive_attention(dev(q), dev(k), dev(v), scale, nbits, phases=3 + valu)
    rtol, atol = kv_tolerance(kv_ref)
    assert_close(host(kv), kv_ref, rtol, atol, "K^T V")
    assert_close(host(out), o_ref, ATTN_RTOL, ATTN_ATOL, "Q(K^T V)")
    # phases run separately give the same bits as the fused call
    _, kv1 = sa.sa_additive_attention(None, dev(k), dev(v), scale, nbits, phases=1 + valu)
    assert torch.equal(kv1, kv)
    out2, _ = sa.sa_additive_attention(dev(q), None, None, scale, nbits, phases=2 + valu, kv=kv1)
    assert torch.equal(out2, out)


def test_additive_attention_wide_range_values(sa):
    """V with magnitudes across 2^-40 .. 2^40 and exact powers of two: the three-term bf16 split must
    carry every fp32 value exactly, so tiny addends are not lost next to large ones of other rows."""
    B, H, N, nbits, dv = 1, 1, 160, 64, 32
    g = np.random.default_rng(11)
    q = wl.random_codes(3, (B, H, N), nbits)
    k = wl.random_codes(4, (B, H, N), nbits)
    v = (g.standard_normal((B, N, H, dv)) * np.exp2(g.integers(-40, 41, size=(B, N, H, 1)))).astype(np.float32)
    v[0, :8, 0, :] = np.exp2(np.arange(8, dtype=np.float32))[:, None]
    o_ref, kv_ref = oracle.additive_attention(q, k, v, nbits, 1.0)
    out, kv = sa.sa_additive_attention(dev(q), dev(k), dev(v), 1.0, nbits)
    rtol, atol = kv_tolerance(kv_ref)
    assert_close(host(kv), kv_ref, rtol, atol, "K^T V, wide range")
    # a single token: K^T V is +-V exactly, whatever the magnitudes
    _, kv1 = sa.sa_additive_attention(None, dev(k[:, :, :1]), dev(v[:, :1]), 1.0, nbits, phases=1)
    bits = ((k[0, 0, 0, 0] >> np.arange(64, dtype=np.uint64)) & np.uint64(1)).astype(np.float64) * 2 - 1
    assert np.array_equal(host(kv1)[0, 0].astype(np.float64), bits[:, None] * v[0, 0, 0].astype(np.float64)[None, :])


def test_additive_attention_is_reproducible(sa):
    B, H, N, nbits, dv = 1, 2, 3000, 128, 64
    q = dev(wl.random_codes(5, (B, H, N), nbits))
    k = dev(wl.random_codes(6, (B, H, N), nbits))
    v = dev(np.random.default_rng(7).standard_normal((B, N, H, dv), dtype=np.float32))
    a, kva = sa.sa_additive_attention(q, k, v, 0.01, nbits)
    b, kvb = sa.sa_additive_attention(q, k, v, 0.01, nbits)
    assert torch.equal(a, b) and torch.equal(kva, kvb)


# --------------------------------------------------------- Hamming attention ----

@pytest.mark.parametrize("B,H,Nq,Nk,nbits,dv,scale", [
    (2, 12, 197, 197, 128, 64, None),   # c4 widths
    (1, 2, 70, 130, 64, 32, None),
    (1, 1, 64, 64, 256, 128, None),
    (1, 2, 33, 50, 128, 64, 3.0),       # sharp softmax -> row-reference path
    (1, 2, 33, 50, 128, 64, -0.2),      # negative scale -> row-reference path
    (1, 1, 5, 1, 64, 64, None),         # one key
    (1, 2, 300, 333, 128, 64, None),    # two query chunks, three key chunks, ragged tails
    (1, 1, 40, 150, 512, 32, None),     # 512-bit codes: popcount scores only
    (1, 1, 70, 200, 256, 64, 2.0),      # 256-bit codes, row-reference path, two key chunks
])
def test_hamming_attention_matches_oracle(sa, B, H, Nq, Nk, nbits, dv, scale):
    q = wl.random_codes(11, (B, H, Nq), nbits)
    k = wl.random_codes(12, (B, H, Nk), nbits)
    v = np.random.default_rng([13, B, H, Nk, dv]).standard_normal((B, Nk, H, dv), dtype=np.float32)
    if scale is None:
        scale = float(np.float32(1.0 / math.sqrt(nbits)))
    ref = oracle.hamming_attention(q, k, v, nbits, scale)
    s_ref = oracle.hamming_scores(q, k, nbits)
    out, scores = sa.sa_hamming_attention(dev(q), dev(k), dev(v), scale, nbits, want_scores=True)
    assert np.array_equal(host(scores), s_ref)
    assert_close(host(out), ref, ATTN_RTOL, ATTN_ATOL, "Hamming attention")
    # scores by XOR + popcount on the vector ALU, and (up to 256 bits) as sign dot products on the matrix cores
    for variant in ((0, 1) if nbits <= 256 else (0,)):
        o2, _, _ = sa.sa_hamming_attention_fused(dev(q), dev(k), dev(v), scale, nbits, 1.0, want_xq=False,
                                                 want_xh=False, variant=variant)
        assert_close(host(o2), ref, ATTN_RTOL, ATTN_ATOL, "Hamming attention, variant %d" % variant)


@pytest.mark.parametrize("B,H,Nq,Nk,nbits,dv", [
    (50, 12, 40, 40, 128, 64),      # 600 units: more than fit the chip at once, so workgroups walk over several
    (33, 12, 70, 150, 64, 64),      # two key chunks per unit, several units per workgroup, ragged tails
    (40, 16, 33, 129, 256, 32),     # a chunk of one key; 256-bit codes; 32-wide heads
    (3, 64, 300, 50, 128, 64),      # two query chunks per (batch, head): 384 units
    (2, 3, 197, 197, 128, 64),      # fewer units than slots: one unit per workgroup
    (9, 8, 100, 113, 128, 64),
    (9, 8, 60, 272, 64, 64),        # three chunks, the last of 16 keys
    (6, 16, 50, 140, 256, 64),      # 256-bit codes at 64-wide heads
    (1, 1, 1, 1, 64, 32),
])
def test_hamming_pipeline_is_bit_identical_to_the_one_unit_kernel(sa, B, H, Nq, Nk, nbits, dv):
    """What sa_hamming_attention runs by default (workgroups that walk over several (batch, head) units with the next
    chunk of V and key codes in flight) against the kernel that takes one unit per workgroup: the same operations in
    the same order, so all three output forms must agree bit for bit; the latter is checked against the oracle above,
    and sampled (batch, head) pairs are checked against it here as well."""
    q = wl.random_codes(21, (B, H, Nq), nbits)
    k = wl.random_codes(22, (B, H, Nk), nbits)
    v = np.random.default_rng([23, B, H, Nk, dv]).standard_normal((B, Nk, H, dv), dtype=np.float32)
    scale = float(np.float32(1.0 / math.sqrt(nbits)))
    dq, dk, dv_ = dev(q), dev(k), dev(v)
    o_pipe, xq_pipe, xh_pipe = sa.sa_hamming_attention_fused(dq, dk, dv_, scale, nbits, 11.0, variant=2)
    o_unit, xq_unit, xh_unit = sa.sa_hamming_attention_fused(dq, dk, dv_, scale, nbits, 11.0, variant=0)
    assert torch.equal(o_pipe, o_unit) and torch.equal(xq_pipe, xq_unit) and torch.equal(xh_pipe, xh_unit)
    # a second call into the same buffers (nothing of the first call's state may matter)
    o_again, _, _ = sa.sa_hamming_attention_fused(dq, dk, dv_, scale, nbits, 11.0, variant=2, want_xq=False, want_xh=False)
    assert torch.equal(o_again, o_unit)
    got = host(o_pipe)
    for b in sorted({0, B // 2, B - 1}):
        ref = oracle.hamming_attention(q[b:b + 1], k[b:b + 1], v[b:b + 1], nbits, scale)
        assert_close(got[b:b + 1], ref, ATTN_RTOL, ATTN_ATOL, "pipelined Hamming attention, batch %d" % b)


# --------------------------------------------------------------- shift layer ----

@pytest.mark.parametrize("variant", [0, 1])
@pytest.mark.parametrize("M,K,N", [
    (300, 384, 1536),     # c3 first layer, ragged M
    (261, 1536, 384),     # c3 second layer
    (129, 192, 768),      # c1 (N and K not multiples of 128)
    (1, 64, 1),           # degenerate
    (64, 3072, 200),      # c4 depth, ragged N
])
def test_shift_linear_bit_exact(sa, variant, M, K, N):
    w4 = wl.shift_weights(3, 4, N, K)
    x = wl.int8_activations(3, M, K)
    ref = oracle.shift_linear(x, w4)
    got = host(sa.sa_shift_linear(dev(x), dev(w4), variant=variant))
    assert np.array_equal(got, ref)


@pytest.mark.parametrize("variant", [0, 1])
def test_shift_linear_extremes_and_bias(sa, variant):
    M, K, N = 70, 128, 130
    x = np.full((M, K), 127, dtype=np.int8)
    x[1::2] = -127
    w4 = np.full((N, K // 2), 0x77, dtype=np.uint8)       # +128 everywhere
    w4[1::2] = 0xFF                                       # -128 everywhere
    bias = (np.arange(N, dtype=np.int32) - 50) * 100000
    ref = oracle.shift_linear(x, w4, bias)
    got = host(sa.sa_shift_linear(dev(x), dev(w4), dev(bias), variant=variant))
    assert np.array_equal(got, ref)


def test_shift_planes_are_the_two_terms_of_the_weight(sa):
    """Prepared planes: A + B == s * 2^e for every weight, both within int8."""
    N, K = 70, 128
    neg, e = wl.shift_weight_raw(3, 6, N, K)
    planes = host(sa.sa_shift_planes_prepare(dev(wl.pack_w4(neg, e)))).astype(np.int64)
    w = np.where(neg == 1, -1, 1) * (1 << e.astype(np.int64))
    assert planes.shape == (2, N, K)
    assert np.array_equal(planes[0] + planes[1], w)
    assert np.abs(planes).max() <= 128 and planes.max() <= 127


@pytest.mark.parametrize("M,K,N", [(300, 384, 1536), (261, 1536, 384), (129, 192, 768), (1, 64, 1), (64, 3072, 200)])
def test_shift_linear_on_prepared_planes(sa, M, K, N):
    w4 = wl.shift_weights(3, 4, N, K)
    x = wl.int8_activations(3, M, K)
    planes = sa.sa_shift_planes_prepare(dev(w4))
    got = host(sa.sa_shift_linear(dev(x), planes, variant=3))
    assert np.array_equal(got, oracle.shift_linear(x, w4))


@pytest.mark.parametrize("seed", range(10))
def test_shift_linear_random_shapes(sa, seed):
    """Ragged M and N around the tile edges of all three int8 tilings (row tiles of 128 and 256, column tiles of
    128, stages of 64 and 128 bytes), weights decoded per call and prepared planes."""
    g = np.random.default_rng([77, seed])
    M = int(g.choice([1, 63, 127, 129, 255, 257, 511, 700, 1025])) + int(g.integers(0, 3))
    K = 32 * int(g.choice([1, 2, 3, 4, 5, 6, 10, 16, 24, 64, 66, 67, 96]))
    N = int(g.choice([1, 31, 127, 128, 129, 200, 383, 640, 1300]))
    neg = g.integers(0, 2, size=(N, K), dtype=np.uint8)
    e = g.integers(0, 8, size=(N, K), dtype=np.uint8)
    w4 = wl.pack_w4(neg, e)
    x = g.integers(-127, 128, size=(M, K), dtype=np.int8)
    ref = oracle.shift_linear(x, w4)
    assert np.array_equal(host(sa.sa_shift_linear(dev(x), dev(w4), variant=1)), ref), (M, K, N)
    planes = sa.sa_shift_planes_prepare(dev(w4))
    assert np.array_equal(host(sa.sa_shift_linear(dev(x), planes, variant=3)), ref), (M, K, N)


@pytest.mark.parametrize("M,K,N", [(40, 96, 33), (3136, 32, 32), (777, 32, 256), (196, 160, 640), (1300, 160, 160),
                                   (130, 224, 129), (257, 32, 1)])
def test_shift_linear_rows_that_end_inside_a_stage(sa, M, K, N):
    """K a multiple of 32 but not of 64: the matrix-core variants pad the weight planes with zeros to whole 64-byte
    stages and read the activation rows as they are (the last stage re-reads bytes from inside the row against
    those zeros).  Every variant, with extreme activations in the last columns and rows."""
    w4 = wl.shift_weights(3, 5, N, K)
    x = wl.int8_activations(3, M, K, extra=5)
    x[-1, :] = 127
    x[:, -1] = -127
    x[0, K - 32:] = 127
    ref = oracle.shift_linear(x, w4)
    planes = sa.sa_shift_planes_prepare(dev(w4))
    assert planes.shape == (2, N, (K + 63) // 64 * 64)
    assert not host(planes)[:, :, K:].any()
    for variant, w in ((0, dev(w4)), (1, dev(w4)), (2, dev(w4)), (3, planes)):
        assert np.array_equal(host(sa.sa_shift_linear(dev(x), w, variant=variant)), ref), variant
    # the last activation row is the last bytes of its buffer: a second call on a buffer that ends there
    tight = dev(x.reshape(-1)).clone().view(M, K)
    assert np.array_equal(host(sa.sa_shift_linear(tight, dev(w4), variant=1)), ref)


# -------------------------------------------------------- quantisation glue ----

def test_fused_attention_outputs_are_the_quantiser_and_the_half_rounding_of_out(sa):
    """The int8 and fp16 forms the Hamming kernel writes beside its fp32 output.  Inside the library
    they must be bit for bit what its quantiser and a half rounding give on that fp32 output; against
    the oracle (which runs on its own attention output) the codes may differ by one step where a value
    sits on a rounding boundary."""
    cfg = wl.scaled_down(wl.C4, B=2)
    q, k, v = wl.qkv(cfg)
    pr, scale = wl.proj(cfg), wl.attention_scale(cfg)
    p = wl.mlp_params(cfg)
    qc, kc = sa.sa_binarize(dev(q), dev(pr), cfg.nbits), sa.sa_binarize(dev(k), dev(pr), cfg.nbits)
    out, xq, xh = sa.sa_hamming_attention_fused(qc, kc, dev(v), scale, cfg.nbits, p.act_inv_scale)
    plain = sa.sa_hamming_attention(qc, kc, dev(v), scale, cfg.nbits)
    assert torch.equal(out, plain)
    # same kernel arithmetic on the same fp32 values: the library's own quantiser must agree exactly
    assert torch.equal(xq, sa.sa_quantize_act(out.view(cfg.T, cfg.E), p.act_inv_scale))
    assert torch.equal(xh, out.view(cfg.T, cfg.E).to(torch.float16))
    # the fp32 output is optional when a narrower form is requested
    none, xq2, _ = sa.sa_hamming_attention_fused(qc, kc, dev(v), scale, cfg.nbits, p.act_inv_scale, want_out=False,
                                                 want_xh=False)
    assert none is None and torch.equal(xq2, xq)
    # and against the oracle end to end: codes differ by at most one step, and rarely
    o_ref = oracle.hamming_attention(oracle.binarize(q, pr, cfg.nbits), oracle.binarize(k, pr, cfg.nbits), v,
                                     cfg.nbits, scale)
    xq_ref = oracle.quantize_act(o_ref.reshape(cfg.T, cfg.E).astype(np.float32), p.act_inv_scale)
    diff = np.abs(host(xq).astype(np.int32) - xq_ref.astype(np.int32))
    assert diff.max() <= 1 and (diff != 0).mean() < 1e-3


def test_quantize_act_half_and_mult_expert_on_half_rows(sa):
    cfg = wl.scaled_down(wl.C1, B=2, N=150)
    p = wl.mlp_params(cfg)
    T, E = cfg.T, cfg.E
    x = wl.float_activations(1, T, E)
    xq, xh = sa.sa_quantize_act_half(dev(x), p.act_inv_scale)
    assert np.array_equal(host(xq), oracle.quantize_act(x, p.act_inv_scale))
    assert np.array_equal(host(xh).astype(np.float64), oracle.round_to_half(x.astype(np.float64)))
    logits = wl.router_logits(cfg)
    perm_r, _, cnt_r, _ = oracle.moe_dispatch(logits)
    rows = perm_r[: cnt_r[0]]
    ref = oracle.mult_mlp(x, rows, p.mw1, p.mw2)
    out = sa.sa_mult_mlp_f16_half(xh, dev(p.mw1), dev(p.mw2), rows=dev(rows))
    assert_close(host(out), ref, 2e-3, 1e-3, "Mult expert on fp16 rows")


def test_quantize_act_bit_exact(sa):
    g = np.random.default_rng(21)
    x = (g.standard_normal(100003) * 3).astype(np.float32)
    x[:16] = [0.5, 1.5, 2.5, -0.5, -1.5, -2.5, 126.5, 127.5, 300.0, -127.5, -1e9, 3.0, -0.0,
              np.nan, np.inf, -np.inf]
    for inv in (1.0, 31.75, 254.0):
        ref = oracle.quantize_act(x, inv)
        assert np.array_equal(host(sa.sa_quantize_act(dev(x), inv)), ref)


def test_requant_lut_bit_exact(sa):
    g = np.random.default_rng(22)
    y = g.integers(-2**31, 2**31, size=50001, dtype=np.int64).astype(np.int32)
    y[:8] = [0, 1, -1, 16777217, -16777217, 2**31 - 1, -2**31, 48]
    lut = wl.activation_lut()
    for s in (1 / 32, 7.0e-4, 1e-7):
        ref = oracle.requant_lut(y, s, lut)
        assert np.array_equal(host(sa.sa_requant_lut(dev(y), s, dev(lut))), ref)


# ------------------------------------------------------------------ dispatch ----

@pytest.mark.parametrize("T,E,tie_every", [(197, 2, 0), (12608, 2, 0), (1000, 2, 7), (3001, 4, 5),
                                           (1, 2, 0), (256, 2, 1), (1023, 8, 3), (1025, 3, 0),
                                           (32768, 2, 3), (32769, 2, 0), (40000, 4, 9),        # either side of the one-launch limit
                                           (131072, 2, 11), (131073, 2, 0), (200001, 8, 5)])   # the last two: the separate scan kernel
def test_moe_dispatch_bit_exact(sa, T, E, tie_every):
    g = np.random.default_rng([31, T, E])
    logits = g.standard_normal((T, E), dtype=np.float32)
    if tie_every:
        logits[::tie_every] = logits[::tie_every, :1]
    perm_r, eo_r, cnt_r, gate_r = oracle.moe_dispatch(logits)
    perm, eo, cnt, gate = sa.sa_moe_dispatch(dev(logits))
    assert np.array_equal(host(cnt), cnt_r)
    assert np.array_equal(host(eo), eo_r)
    assert np.array_equal(host(perm), perm_r)
    assert_close(host(gate), gate_r, 1e-6, 0.0, "gate")


@pytest.mark.parametrize("cfg", [wl.C1, wl.C4])
def test_moe_dispatch_on_the_config_router(sa, cfg):
    logits = wl.router_logits(cfg)
    perm_r, eo_r, cnt_r, _ = oracle.moe_dispatch(logits)
    perm, eo, cnt, _ = sa.sa_moe_dispatch(dev(logits))
    assert np.array_equal(host(cnt), cnt_r) and np.array_equal(host(perm), perm_r)
    assert np.array_equal(np.sort(host(perm)), np.arange(cfg.T))


# ------------------------------------------------------------------- experts ----

@pytest.mark.parametrize("variant", [0, 1])
def test_shift_mlp_bit_exact_with_row_lists(sa, variant):
    cfg = wl.scaled_down(wl.C1, B=2, N=150)
    p = wl.mlp_params(cfg)
    T, E = cfg.T, cfg.E
    xq = wl.int8_activations(1, T, E)
    logits = wl.router_logits(cfg)
    perm_r, _, cnt_r, gate_r = oracle.moe_dispatch(logits)
    rows = perm_r[cnt_r[0]:]
    y2_ref = oracle.shift_mlp(xq[rows], p.w1, p.w2, p.requant_scale, p.lut)
    d_xq, d_w1, d_w2, d_lut = dev(xq), dev(p.w1), dev(p.w2), dev(p.lut)
    # (a) explicit row list
    y2 = sa.sa_shift_mlp(d_xq, d_w1, d_w2, p.requant_scale, d_lut, rows=dev(rows), variant=variant)
    assert np.array_equal(host(y2), y2_ref)
    # (b) device-side segment of a dispatch result + gated scatter
    perm, _, cnt, gate = sa.sa_moe_dispatch(dev(logits))
    y = torch.zeros((T, E), dtype=torch.float32, device="cuda")
    y2b = sa.sa_shift_mlp(d_xq, d_w1, d_w2, p.requant_scale, d_lut, rows=perm, counts=cnt, expert=1,
                          max_rows=T, y=y, gate=gate, out_scale=p.out_scale, variant=variant)
    assert np.array_equal(host(y2b)[: rows.size], y2_ref)
    y_ref = np.zeros((T, E))
    y_ref[rows] = gate_r[rows, None] * (np.float64(np.float32(p.out_scale)) * y2_ref)
    assert_close(host(y), y_ref, 2e-6, 1e-30, "shift expert scatter")
    # (c) all rows, no list
    y2c = sa.sa_shift_mlp(d_xq, d_w1, d_w2, p.requant_scale, d_lut, variant=variant)
    assert np.array_equal(host(y2c), oracle.shift_mlp(xq, p.w1, p.w2, p.requant_scale, p.lut))
    # (d) weights decoded beforehand
    if variant == 1:
        y2d = sa.sa_shift_mlp(d_xq, sa.sa_shift_planes_prepare(d_w1), sa.sa_shift_planes_prepare(d_w2),
                              p.requant_scale, d_lut, rows=dev(rows), variant=3)
        assert np.array_equal(host(y2d), y2_ref)


@pytest.mark.parametrize("scale", [0.5, 1.0, -0.25, 1e-9, 1e30, float("inf"), float("-inf"), float("nan"), 0.0])
def test_shift_mlp_requant_scale_edge_cases(sa, scale):
    """The fused requantisation between the two Shift layers: ties (scale 0.5 on odd sums), saturation,
    sign flip, and the non-finite scales (NaN -> code 0 everywhere; Inf saturates, and 0 * Inf -> code 0)."""
    cfg = wl.scaled_down(wl.C1, B=1, N=70)
    p = wl.mlp_params(cfg)
    xq = wl.int8_activations(1, cfg.T, cfg.E, extra=9)
    xq[0, :] = 0                                              # an all-zero row: 0 * Inf
    ref = oracle.shift_mlp(xq, p.w1, p.w2, scale, p.lut)
    for variant in (0, 1):
        got = sa.sa_shift_mlp(dev(xq), dev(p.w1), dev(p.w2), scale, dev(p.lut), variant=variant)
        assert np.array_equal(host(got), ref), "variant %d" % variant


def test_mult_mlp_matches_oracle(sa):
    cfg = wl.scaled_down(wl.C1, B=2, N=150)
    p = wl.mlp_params(cfg)
    T, E = cfg.T, cfg.E
    x = wl.float_activations(1, T, E)
    logits = wl.router_logits(cfg)
    perm_r, _, cnt_r, gate_r = oracle.moe_dispatch(logits)
    rows = perm_r[: cnt_r[0]]
    ref = oracle.mult_mlp(x, rows, p.mw1, p.mw2)
    d_x, d_w1, d_w2 = dev(x), dev(p.mw1), dev(p.mw2)
    out = sa.sa_mult_mlp_f16(d_x, d_w1, d_w2, rows=dev(rows))
    assert_close(host(out), ref, 2e-3, 1e-3, "Mult expert")
    perm, _, cnt, gate = sa.sa_moe_dispatch(dev(logits))
    y = torch.zeros((T, E), dtype=torch.float32, device="cuda")
    sa.sa_mult_mlp_f16(d_x, d_w1, d_w2, rows=perm, counts=cnt, expert=0, max_rows=T, want_out=False,
                       y=y, gate=gate)
    y_ref = np.zeros((T, E))
    y_ref[rows] = gate_r[rows, None] * ref
    assert_close(host(y), y_ref, 2e-3, 1e-3, "Mult expert scatter")


def test_gather_and_combine_rows(sa):
    T, E = 500, 64
    g = np.random.default_rng(41)
    src = g.standard_normal((T, E), dtype=np.float32)
    rows = g.permutation(T)[:123].astype(np.int32)
    got = host(sa.sa_gather_rows(dev(src), rows=dev(rows)))
    assert np.array_equal(got, src[rows])
    gate = g.uniform(0.5, 1.0, T).astype(np.float32)
    y = torch.zeros((T, E), dtype=torch.float32, device="cuda")
    sa.sa_combine_rows(dev(src[:123]), y, rows=dev(rows), gate=dev(gate))
    ref = np.zeros((T, E), dtype=np.float32)
    ref[rows] = gate[rows, None] * src[:123]
    assert np.array_equal(host(y), ref)


# --------------------------------------------------------------------- block ----

def _block_inputs(cfg):
    q, k, v = wl.qkv(cfg)
    pr = wl.proj(cfg)
    scale = wl.attention_scale(cfg)
    p = wl.mlp_params(cfg) if cfg.E else None
    logits = wl.router_logits(cfg) if (cfg.E and cfg.shift_frac is not None) else None
    return q, k, v, pr, scale, p, logits


def run_block(sa, cfg, inputs, prepared=False):
    """prepared: the Shift weights enter as planes decoded beforehand (what bench.py times)."""
    q, k, v, pr, scale, p, logits = inputs
    kw = dict(B=cfg.B, N=cfg.N, H=cfg.H, d=cfg.d, nbits=cfg.nbits, dv=cfg.dv,
              attention=0 if cfg.attention == "linear" else 1, hid=cfg.hid, moe=logits is not None,
              attn_scale=scale, q=dev(q), k=dev(k), v=dev(v), proj=dev(pr))
    if p is not None:
        w1, w2 = dev(p.w1), dev(p.w2)
        if prepared:
            w1, w2 = sa.sa_shift_planes_prepare(w1), sa.sa_shift_planes_prepare(w2)
            kw.update(shift_variant=3)
        kw.update(act_inv_scale=p.act_inv_scale, requant_scale=p.requant_scale, out_scale=p.out_scale,
                  w1=w1, w2=w2, lut=dev(p.lut))
        if logits is not None:
            kw.update(logits=dev(logits), mw1=dev(p.mw1), mw2=dev(p.mw2))
    blk = sa.binding.Block(**kw)
    o, y = blk.forward()
    torch.cuda.synchronize()
    return host(o), (None if y is None else host(y))


def check_block_output(y, y_ref):
    """End-to-end MLP output.  The fp32 attention output feeds an int8 quantiser whose step is
    1/inv_scale, about 1/32 of the rms of its input.  The attention output carries a relative
    error of a few 1e-6 (bf16 three-product P*V of the Hamming kernel; ~1e-5 absolute at N = 16384
    for the linear kernel), so an element lands on the other side of a rounding boundary with
    probability ~1e-4, and a token of E = 256..768 elements carries at least one flipped code with
    probability up to ~10 %.  One flipped code shifts every fc1 accumulator of that token by 2^e,
    flips a few dozen hidden codes and moves that token's outputs by ~1e-2 of the output rms.  So
    the test asks: at least 90 % of the outputs agree to float accuracy, and none is further than
    5e-2 rms away.  Stage-level tests on shared inputs carry the bit-exact claims."""
    rms = float(np.sqrt(np.mean(np.square(y_ref))))
    err = np.abs(y.astype(np.float64) - y_ref)
    tight = err <= 2e-3 * np.abs(y_ref) + 1e-3 * rms
    assert tight.mean() > 0.90, "only %.4f of the block outputs agree tightly" % tight.mean()
    assert err.max() <= 5e-2 * rms, "worst block output error %.3g (rms %.3g)" % (err.max(), rms)


@pytest.mark.parametrize("cfg", [
    wl.C1,
    wl.scaled_down(wl.C2, B=2, N=700),
    wl.scaled_down(wl.C4, B=2),
    wl.scaled_down(wl.C5, B=1, N=1100),
], ids=lambda c: c.name)
def test_block_forward_matches_oracle(sa, cfg):
    inputs = _block_inputs(cfg)
    q, k, v, pr, scale, p, logits = inputs
    o_ref, y_ref = oracle.block_forward(cfg, q, k, v, pr, scale, logits, p)
    o, y = run_block(sa, cfg, inputs)
    assert_close(o, o_ref, ATTN_RTOL, ATTN_ATOL, "attention output")
    if y_ref is not None:
        check_block_output(y, y_ref)
        # the same block on Shift weights decoded beforehand: the same kernels on the same planes
        o2, y2 = run_block(sa, cfg, inputs, prepared=True)
        assert np.array_equal(o2, o) and np.array_equal(y2, y)


# ------------------------- {0,1} codes with the row normaliser, depthwise conv ----

@pytest.mark.parametrize("valu", [0, 4], ids=["mfma", "valu"])
@pytest.mark.parametrize("B,H,Nq,Nk,nbits,dv", [
    (2, 3, 197, 197, 64, 64),      # c1 widths
    (2, 1, 700, 700, 64, 32),      # c2 widths, ragged token tail
    (1, 4, 1100, 1100, 256, 64),   # c5 widths
    (1, 2, 70, 333, 128, 128),     # Nq != Nk, dv = 128
    (1, 1, 5, 1, 64, 32),          # a single key
    (1, 2, 300, 300, 192, 64),     # three words: VALU second phase
])
def test_linear_attention_01_matches_oracle(sa, B, H, Nq, Nk, nbits, dv, valu):
    g = np.random.default_rng([81, Nq, Nk, nbits])
    qc = wl.random_codes(5, (B, H, Nq), nbits)
    kc = wl.random_codes(6, (B, H, Nk), nbits)
    qc[0, 0, 0] = 0                                              # a query that selects nothing
    v = g.standard_normal((B, Nk, H, dv)).astype(np.float32)
    eps = 1.0
    ref, kv_ref, ksum_ref, den_ref = oracle.linear_attention_01(qc, kc, v, nbits, eps)
    out, kv, ksum = sa.sa_linear_attention_01(dev(qc), dev(kc), dev(v), eps, nbits, phases=3 | valu)
    assert np.array_equal(host(ksum).astype(np.int64), ksum_ref)
    assert_close(host(kv), kv_ref, *kv_tolerance(kv_ref), "{0,1} K^T V")
    assert_close(host(out), ref, ATTN_RTOL, ATTN_ATOL, "normalised linear attention")
    assert np.all(host(out)[0, 0, 0] == 0.0)
    # the two phases separately give the same bits
    _, kv1, ksum1 = sa.sa_linear_attention_01(None, dev(kc), dev(v), eps, nbits, phases=1 | valu)
    out2, _, _ = sa.sa_linear_attention_01(dev(qc), None, None, eps, nbits, phases=2 | valu, kv=kv1, ksum=ksum1)
    assert torch.equal(out2, out)


@pytest.mark.parametrize("B,gh,gw,E", [(2, 14, 14, 192), (1, 56, 56, 32), (3, 5, 7, 12), (1, 1, 9, 64), (1, 4, 3, 1028)])
def test_dwconv3x3_matches_oracle(sa, B, gh, gw, E):
    g = np.random.default_rng([82, gh, gw, E])
    v = g.standard_normal((B, gh, gw, E)).astype(np.float32)
    w = g.standard_normal((E, 3, 3)).astype(np.float32)
    bias = g.standard_normal(E).astype(np.float32)
    ref = oracle.dwconv3x3(v, w, bias)
    assert_close(host(sa.sa_dwconv3x3(dev(v), dev(w), dev(bias))), ref, 1e-5, 1e-5, "depthwise conv")
    base = g.standard_normal((B, gh, gw, E)).astype(np.float32)
    got = host(sa.sa_dwconv3x3(dev(v), dev(w), None, out=dev(base), accumulate=True))
    assert_close(got, oracle.dwconv3x3(v, w) + base.astype(np.float64), 1e-5, 1e-5, "depthwise conv added to an output")


# ------------------------------------------------ balancing loss (Eq. 4), forward ----

@pytest.mark.parametrize("T,E,sigma", [(197, 2, 0.1), (12608, 2, 0.05), (3001, 4, 0.02), (1000, 8, 0.2), (1, 2, 1.0)])
def test_moe_balance_loss_matches_oracle(sa, T, E, sigma):
    logits = np.random.default_rng([83, T, E]).standard_normal((T, E)).astype(np.float32)
    alpha = (np.arange(E, 0, -1) / np.arange(E, 0, -1).sum()).astype(np.float32)
    ref_losses, ref_sums = oracle.moe_balance_loss(logits, alpha, sigma)
    losses, sums = sa.sa_moe_balance_loss(dev(logits), dev(alpha), sigma)
    assert_close(host(sums), ref_sums, 2e-5, 1e-6, "importance / load sums")
    assert_close(host(losses), ref_losses, 2e-4, 1e-7, "L_IMP, L_LOAD")


def test_moe_balance_loss_on_the_config_router(sa):
    """Config 4's constructed router: 70 % of the tokens favour the Shift expert; with alpha = (0.7, 0.3)
    (Mult : Shift latency 7 : 3) the weighted loads are nearly flat and L_LOAD is near 0."""
    logits = wl.router_logits(wl.C4)
    alpha = np.array([0.7, 0.3], dtype=np.float32)
    ref_losses, ref_sums = oracle.moe_balance_loss(logits, alpha, 0.01)
    losses, sums = sa.sa_moe_balance_loss(dev(logits), dev(alpha), 0.01)
    assert_close(host(sums), ref_sums, 2e-5, 1e-6, "sums")
    assert_close(host(losses), ref_losses, 2e-4, 1e-7, "losses")
    assert ref_losses[1] < 1e-3


def test_block_forward_replays_from_a_captured_graph(sa):
    """The block enqueues kernels on the caller's stream only (buffers are cleared by kernels, not by memset
    nodes), so a caller may capture it.  Every replay, with eager
    work and synchronisations in between, must reproduce the eager result bit for bit."""
    cfg = wl.scaled_down(wl.C4, B=3)
    q, k, v, pr, scale, p, logits = _block_inputs(cfg)
    kw = dict(B=cfg.B, N=cfg.N, H=cfg.H, d=cfg.d, nbits=cfg.nbits, dv=cfg.dv, attention=1, hid=cfg.hid, moe=True,
              attn_scale=scale, q=dev(q), k=dev(k), v=dev(v), proj=dev(pr), act_inv_scale=p.act_inv_scale,
              requant_scale=p.requant_scale, out_scale=p.out_scale, w1=dev(p.w1), w2=dev(p.w2), lut=dev(p.lut),
              logits=dev(logits), mw1=dev(p.mw1), mw2=dev(p.mw2))
    blk = sa.binding.Block(**kw)
    o, y = blk.forward()
    torch.cuda.synchronize()
    o_ref, y_ref = o.clone(), y.clone()
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.stream(side):
        blk.forward()
        torch.cuda.synchronize()
        graph.capture_begin()
        blk.forward()
        graph.capture_end()
    torch.cuda.synchronize()
    for rep in range(4):
        o.zero_()
        y.zero_()
        if rep % 2:
            blk.forward()                          # eager work between replays
            o.zero_()
            y.zero_()
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(o, o_ref) and torch.equal(y, y_ref), "replay %d" % rep


def test_block_forward_on_two_streams_in_turn_is_bit_identical(sa):
    """Successive blocks enqueued on two streams in turn (what bench.py does by default) overlap on the GPU;
    every block must still produce what it produces alone."""
    cfg = wl.scaled_down(wl.C4, B=8)
    q, k, v, pr, scale, p, logits = _block_inputs(cfg)
    g = np.random.default_rng(77)
    blocks, refs = [], []
    for i in range(4):
        qi = (q + np.float32(0.01 * i) * g.standard_normal(q.shape, dtype=np.float32)).astype(np.float32)
        kw = dict(B=cfg.B, N=cfg.N, H=cfg.H, d=cfg.d, nbits=cfg.nbits, dv=cfg.dv, attention=1, hid=cfg.hid, moe=True,
                  attn_scale=scale, q=dev(qi), k=dev(k), v=dev(v), proj=dev(pr), act_inv_scale=p.act_inv_scale,
                  requant_scale=p.requant_scale, out_scale=p.out_scale, w1=dev(p.w1), w2=dev(p.w2), lut=dev(p.lut),
                  logits=dev(logits), mw1=dev(p.mw1), mw2=dev(p.mw2))
        blk = sa.binding.Block(**kw)
        o, y = blk.forward()
        torch.cuda.synchronize()
        blocks.append(blk)
        refs.append((o.clone(), y.clone()))
    streams = [torch.cuda.Stream(), torch.cuda.Stream()]
    for rep in range(3):
        for blk in blocks:
            blk.o.zero_()
            blk.y.zero_()
        torch.cuda.synchronize()
        for i in range(16):
            with torch.cuda.stream(streams[i % 2]):
                blocks[i % 4].forward()
        torch.cuda.synchronize()
        for blk, (o_ref, y_ref) in zip(blocks, refs):
            assert torch.equal(blk.o, o_ref) and torch.equal(blk.y, y_ref), "rep %d" % rep


# ------------------------------------------------------- MoE form of a Linear ----

@pytest.mark.parametrize("variant", [0, 1, 3], ids=["valu", "mfma", "prepared"])
@pytest.mark.parametrize("T,K,N,shift_frac", [
    (1576, 768, 768, 0.7),        # a DeiT-Base attention Linear on 8 images
    (300, 192, 576, 0.5),         # DeiT-Tiny Q/K/V width, ragged row tiles
    (777, 160, 160, 0.9),         # K not a multiple of 64: the padded last stage
    (64, 32, 20, 0.0),            # every token to the Mult expert; N not a multiple of 4 chunks
    (65, 64, 36, 1.0),            # every token to the Shift expert
    (40000, 64, 32, 0.6),         # more tokens than the one-launch routing takes
    (1, 32, 4, 0.5),
])
def test_moe_linear_matches_oracle(sa, variant, T, K, N, shift_frac):
    """Sec. 4.1's MoE option for a Linear layer.  Routing and gate bit-exact / 1e-6; Shift rows are exact integers
    times two fp32 factors (relative 3e-7 covers the two roundings); Mult rows carry fp32 accumulation of fp16
    products (2e-3 relative to the row scale, as for the Mult expert of the MLP)."""
    g = np.random.default_rng([17, T, K, N])
    x = (g.standard_normal((T, K)) * 2).astype(np.float32)
    # logits whose second entry exceeds the first for about shift_frac of the tokens
    margin = g.standard_normal(T).astype(np.float32)
    cut = np.quantile(margin, 1.0 - shift_frac) if 0.0 < shift_frac < 1.0 else (np.inf if shift_frac == 0.0 else -np.inf)
    base = g.standard_normal(T).astype(np.float32)
    logits = np.stack([base, base + np.where(margin > cut, 1.0, -1.0) * (0.1 + np.abs(margin))], axis=1).astype(np.float32)
    neg = g.integers(0, 2, size=(N, K), dtype=np.uint8)
    e = g.integers(0, 8, size=(N, K), dtype=np.uint8)
    w4 = wl.pack_w4(neg, e)
    w_half = (g.standard_normal((N, K)) / np.sqrt(K)).astype(np.float16)
    inv, out_scale = 20.0, 1.0 / (128.0 * K)
    ref = oracle.moe_linear(x, logits, w4, w_half, inv, out_scale)
    _, expert_ref, counts_ref, gate_ref = oracle.moe_dispatch(logits)
    xq = dev(oracle.quantize_act(x, inv))
    xh = dev(x.astype(np.float16))
    d_w = dev(w4)
    if variant == 3:
        d_w = sa.sa_shift_planes_prepare(d_w)
    y, expert_of, gate = sa.sa_moe_linear(xq, xh, dev(logits), d_w, dev(w_half), out_scale, variant=variant, want_routing=True)
    assert np.array_equal(host(expert_of), expert_ref)
    assert np.allclose(host(gate), gate_ref, rtol=1e-6, atol=0)
    got = host(y).astype(np.float64)
    shift_rows, mult_rows = expert_ref == 1, expert_ref == 0
    assert int(shift_rows.sum()) == int(counts_ref[1])
    if shift_rows.any():
        err = np.abs(got[shift_rows] - ref[shift_rows])
        assert np.all(err <= 3e-7 * np.abs(ref[shift_rows]) + 1e-30), "Shift rows: %g" % err.max()
    if mult_rows.any():
        rms = float(np.sqrt(np.mean(ref[mult_rows] ** 2)))
        err = np.abs(got[mult_rows] - ref[mult_rows])
        assert np.all(err <= 2e-3 * np.abs(ref[mult_rows]) + 1e-3 * rms), "Mult rows: %g (rms %g)" % (err.max(), rms)


# ------------------------------------------------------------ measurement helper ----

def test_probe_runs_and_reports_its_clock(sa):
    """sa_probe_mfma is not a step of the path; the check is that it runs, takes the time its instruction count
    implies within wide bounds, and reports a plausible shader clock."""
    out = sa.sa_probe_mfma(0, 2, 8, 2000)
    torch.cuda.synchronize()
    cycles, ticks = int(out[0]), int(out[1])
    assert cycles > 2000 * 8 * 16 and ticks > 0                      # at least 16 cycles per instruction
    assert 500.0 < cycles / ticks * 100.0 < 3500.0                    # MHz
    with pytest.raises(sa.SAError):
        sa.sa_probe_mfma(1, 2, 8, 10)                                 # Shift-like operands are int8 only


# few rows, many outputs: one row as a column of tokens (a last strip of one to four), two rows, a strip that is not full
@pytest.mark.parametrize("B,gh,gw,E", [(1, 1, 8193, 128), (5, 1, 6555, 32), (2, 1, 4098, 132), (3, 2, 1401, 128), (1, 3, 2741, 132), (7, 5, 937, 32)])
def test_dwconv3x3_of_few_rows(sa, B, gh, gw, E):
    test_dwconv3x3_matches_oracle(sa, B, gh, gw, E)


# four outputs below each other in a last strip of one to four rows, one column of tokens, either side of the 2^18 items it takes
@pytest.mark.parametrize("B,gh,gw,E", [(9, 57, 33, 64), (9, 58, 61, 64), (4, 63, 66, 64), (1, 64, 64, 256), (1, 64, 63, 256), (1, 8193, 1, 128),
                                       (8193, 1, 1, 128), (2, 4099, 1, 132)])
def test_dwconv3x3_in_strips(sa, B, gh, gw, E):
    test_dwconv3x3_matches_oracle(sa, B, gh, gw, E)
