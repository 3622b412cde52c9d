"""A call that is refused has launched nothing: on a host without a GPU every bad argument of the composed entry points comes
back with its own code, where a launch before the check would come back as SA_ERR_HIP."""
import ctypes

import pytest
import torch

from paper_2306_06446_amd import binding

FAKE, ODD = 0x1000, 0x1004
INVALID, SHAPE, ALIGN, HIP, UNSUPPORTED = -1, -2, -3, -5, -6


@pytest.fixture(scope="module")
def lib():
    if torch.cuda.device_count() > 0:
        pytest.skip("the pointers of these calls are made up: for hosts without a GPU")
    return binding.load_library()


def block(**kw):
    d = binding.SaBlockDesc(B=2, N=50, H=2, d=64, nbits=128, dv=64, attention=0, hid=256, moe=0, shift_variant=2,
                            attn_scale=0.1, act_inv_scale=1.0, requant_scale=1.0, out_scale=1.0)
    for n in ("q", "k", "v", "proj", "logits", "w1", "w2", "lut", "mw1", "mw2", "o", "y", "workspace"):
        setattr(d, n, FAKE)
    return with_values(d, kw)


def layer(**kw):
    d = binding.SaLayerDesc(B=2, N=50, H=2, nbits=128, E=128, hid=256, attention=0, moe=0, shift_variant=2, eps=1e-6,
                            ln_inv_scale=1.0, qkv_scale=1.0, attn_scale=0.1, act_inv_scale=1.0, o_scale=1.0, requant_scale=1.0,
                            out_scale=1.0)
    for n in ("x", "gamma1", "beta1", "gamma2", "beta2", "wqkv", "wo", "proj", "wg", "bg", "w1", "w2", "lut", "mw1", "mw2", "y",
              "workspace"):
        setattr(d, n, FAKE)
    return with_values(d, kw)


def with_values(d, kw):
    for n, v in kw.items():
        setattr(d, n, v)
    d.workspace_bytes = 1 << 60
    return d


BLOCK_KINDS = [dict(attention=a, moe=m, shift_variant=v, **size) for a in (0, 1) for m in (0, 1) for v in (0, 2, 3)
               for size in (dict(), dict(B=1000))]           # 100 tokens, and more than the one-launch routing takes
LAYER_KINDS = BLOCK_KINDS + [dict(k, proj=None, nbits=64) for k in BLOCK_KINDS]        # the sign hash in the projection's epilogue


@pytest.mark.parametrize("kind", BLOCK_KINDS, ids=str)
def test_block(lib, kind):
    call = lambda **kw: lib.sa_block_forward(ctypes.byref(block(**{**kind, **kw})), None)     # noqa: E731
    assert call() == HIP                                     # nothing to refuse: it goes as far as a launch
    for name in ["q", "k", "v", "proj", "o", "w1", "w2", "lut", "y"] + ["logits", "mw1", "mw2"] * kind["moe"]:
        assert call(**{name: ODD}) == ALIGN, name
    assert call(d=48) == UNSUPPORTED
    assert call(proj=None) == SHAPE                          # 128 bits of 64 features
    assert call(nbits=8192) in (SHAPE, UNSUPPORTED)
    assert call(dv=48) in (UNSUPPORTED, SHAPE)
    assert call(dv=48, hid=0, moe=0) == UNSUPPORTED
    assert call(B=1 << 16, N=1, H=16) == SHAPE               # 2^20 heads
    assert call(hid=96) == SHAPE
    assert call(shift_variant=7) == INVALID
    if kind["attention"] == 1:
        assert call(attn_scale=float("nan")) == INVALID
        assert call(nbits=192) == UNSUPPORTED
    if kind["shift_variant"] == 0:
        assert call(B=1 << 14, N=33) == SHAPE                # more row tiles than a grid of the vector-ALU kernel


@pytest.mark.parametrize("kind", LAYER_KINDS, ids=str)
def test_layer(lib, kind):
    call = lambda **kw: lib.sa_layer_forward(ctypes.byref(layer(**{**kind, **kw})), None)     # noqa: E731
    assert call() == HIP
    names = ["x", "gamma1", "beta1", "gamma2", "beta2", "wqkv", "wo", "w1", "w2", "lut", "y"] + ["wg", "bg", "mw1", "mw2"] * kind["moe"]
    for name in names + ["proj"] * ("proj" not in kind):
        assert call(**{name: ODD}) == ALIGN, name
    assert call(E=256 * 48, H=256) == UNSUPPORTED            # rows of LayerNorm
    assert call(E=192, H=4) in (UNSUPPORTED, SHAPE)          # heads of 48
    assert call(proj=None, nbits=192) in (UNSUPPORTED, SHAPE)
    assert call(B=1 << 18, N=1, H=4, E=256) == SHAPE         # 2^20 heads
    if kind["attention"] == 1:
        assert call(attn_scale=float("inf")) == INVALID


def test_moe_linear_rows_of_the_vector_alu_variant(lib):
    args = [FAKE, FAKE, FAKE, ctypes.c_long(65536 * 8), 64, 64, FAKE, FAKE, ctypes.c_float(1.0), FAKE, None, None, 0, FAKE]
    args = [ctypes.c_void_p(a) if a == FAKE else a for a in args]
    assert lib.sa_moe_linear(*args, ctypes.c_size_t(1 << 60), None) == SHAPE


def test_hamming_score_dump(lib):
    p = ctypes.c_void_p(FAKE)
    assert lib.sa_hamming_attention(p, p, p, p, 1 << 10, 1, 1 << 15, 1 << 15, 64, 64, ctypes.c_float(0.1), p, None) == SHAPE
    assert lib.sa_hamming_attention(p, p, p, p, 1, 1, 4, 4, 192, 64, ctypes.c_float(0.1), p, None) == UNSUPPORTED
