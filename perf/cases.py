"""What a user of this library has it do, as cases that can be timed one by one.

Every case goes through the public entry points of `paper_2306_06446_amd.binding` the way a program that serves or
evaluates a ShiftAddViT model calls them: the weights, the output buffers and the workspace are made once, a pass is one
call (or the two or three calls that belong together).  Widths, token counts and code lengths are those of this
repository's benchmark configurations and of the pyramid-ViT stages its kernel sweep walks over (DeiT-Tiny / Small / Base,
PVT-like stages, a long-range sequence); batch sizes go from one image to the full batches of those configurations.
"""
from __future__ import annotations

import math
import random

import torch

from paper_2306_06446_amd import binding as sa
from paper_2306_06446_amd import workloads as wl

# (E, H, hid, N) of the models whose blocks are run: width, heads, MLP width, tokens of one image or sequence.
_MODELS = {
    "deit-tiny": (192, 3, 768, 197),
    "deit-small": (384, 6, 1536, 197),
    "deit-base": (768, 12, 3072, 197),
    "pvt-stage2": (64, 2, 512, 784),
    "pvt-stage4": (256, 8, 1024, 49),
    "long-seq": (256, 4, 1024, 16384),
}


def _block(name, B, N, H, d, nbits, attention, hid, moe, prepared, shift_frac=0.7):
    """sa_block_forward: hash, attention and (hid > 0) the MLP on Q, K, V that the caller already has."""
    return dict(name=name, kind="block", B=B, N=N, H=H, d=d, nbits=nbits, attention=attention, hid=hid, moe=moe,
                prepared=prepared, shift_frac=shift_frac)


def _layer(name, B, N, H, E, nbits, attention, hid, moe, sign_hash, prepared, shift_frac=0.7):
    """sa_layer_forward: the complete block, from tokens to tokens."""
    return dict(name=name, kind="layer", B=B, N=N, H=H, E=E, nbits=nbits, attention=attention, hid=hid, moe=moe,
                sign_hash=sign_hash, prepared=prepared, shift_frac=shift_frac)


def listed():
    return [
        # one image through a DeiT-Tiny block with its two-expert MLP: the latency of an interactive caller
        _block("tiny block, one image", 1, 197, 3, 64, 64, "linear", 768, True, False, 0.5),
        # the same model's complete block (norms, the four attention Linears, router), weights laid out once
        _layer("tiny layer, one image", 1, 197, 3, 192, 64, "linear", 768, True, False, True, 0.5),
        # attention alone at a pyramid ViT's first stage, batch 32 (56 x 56 tokens, narrow heads)
        _block("pvt stage 1 attention", 32, 3136, 1, 32, 64, "linear", 0, False, False),
        # the same stage with {0,1} codes, the row normaliser and the depthwise convolution on V
        dict(name="pvt stage 1, 0/1 codes + conv", kind="conv01", B=32, gh=56, gw=56, H=1, d=32, nbits=64),
        # a pyramid ViT's second stage as a complete layer, batch 32, every token through the Shift MLP
        _layer("pvt stage 2 layer", 32, 784, 2, 64, 64, "linear", 512, False, False, True),
        # the two Linears of a DeiT-Small MLP as Shift layers with integer outputs, batch 64, packed weights
        dict(name="small shift linears", kind="linears", M=64 * 197, E=384, hid=1536),
        # a few requests at once: DeiT-Base complete layer with the sign hash, batch 7 (an odd number of rows)
        _layer("base layer, sign hash, batch 7", 7, 197, 12, 768, 64, "hamming", 3072, True, True, True),
        # the headline configuration: DeiT-Base block, Hamming attention, MoE 70 / 30, batch 64, packed weights
        _block("base block", 64, 197, 12, 64, 128, "hamming", 3072, True, False),
        # the complete DeiT-Base layer at the same batch, hash by projection, weights laid out once
        _layer("base layer", 64, 197, 12, 768, 128, "hamming", 3072, True, False, True),
        # one Linear of the attention module as a mixture of a Mult and a Shift expert, batch 64
        dict(name="moe linear", kind="moe_linear", T=64 * 197, K=768, N=768, shift_frac=0.7),
        # one long sequence through the complete layer: few heads, many tokens
        _layer("long layer, one sequence", 1, 16384, 4, 256, 256, "linear", 1024, False, False, True),
        # eight long sequences through the block: the largest pass
        _block("long block", 8, 16384, 4, 64, 256, "linear", 1024, False, False),
    ]


def _log_int(rng: random.Random, lo: int, hi: int) -> int:
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _cost(case):
    w = work(case)
    return max(w["bytes"], w["flops"] / 50)


def draw(rng: random.Random):
    """A case of the same ranges: any of the models, batches from one image up, token counts around the models' own."""
    top = max(_cost(c) for c in listed())
    while True:
        kind = rng.choice(("block", "block", "layer", "layer", "attention", "conv01", "linears", "moe_linear"))
        E, H, hid, n_tok = _MODELS[rng.choice(sorted(_MODELS))]
        d = E // H
        attention = "hamming" if n_tok <= 1024 and rng.random() < 0.5 else "linear"
        N = max(2, _log_int(rng, n_tok // 4 if n_tok > 1024 else n_tok // 2, n_tok + n_tok // 2))
        B = _log_int(rng, 1, max(1, min(128, 200000 // N)))
        nbits = rng.choice((64, 128, 256)) if d == 64 else 64
        moe, prepared = rng.random() < 0.5, rng.random() < 0.5
        frac = rng.choice((0.3, 0.5, 0.7))
        if kind == "block":
            case = _block("", B, N, H, d, nbits, attention, hid, moe, prepared, frac)
        elif kind == "layer":
            case = _layer("", B, N, H, E, nbits, attention, hid, moe, nbits == d and rng.random() < 0.5, prepared, frac)
        elif kind == "attention":
            case = _block("", B, N, H, d, nbits, attention, 0, False, False)
        elif kind == "conv01":
            side = max(2, int(math.sqrt(N)))
            case = dict(kind="conv01", B=B, gh=side, gw=max(1, N // side), H=H, d=d, nbits=nbits)
        elif kind == "linears":
            case = dict(kind="linears", M=B * N, E=E, hid=hid)
        else:
            case = dict(kind="moe_linear", T=B * N, K=E, N=rng.choice((E, 3 * E)), shift_frac=frac)
        case.pop("name", None)
        if _cost(case) <= top:
            return case


# ------------------------------------------------------------------------------------------ inputs --

def _randn(g, *shape, std=1.0, dtype=torch.float32):
    return (torch.randn(shape, generator=g, device="cuda", dtype=torch.float32) * std).to(dtype)


def _w4(g, n, k):
    """Packed 4-bit shift weights: sign and exponent uniform, as the repository's synthetic workloads draw them."""
    return torch.randint(0, 256, (n, k // 2), generator=g, device="cuda", dtype=torch.uint8)


def _int8(g, m, k):
    return torch.randint(-127, 128, (m, k), generator=g, device="cuda", dtype=torch.int8)


def _logits(g, T, shift_frac):
    """Router logits of which round(shift_frac * T) favour the Shift expert, with margins of at least 0.01."""
    margin = torch.randn(T, generator=g, device="cuda").abs() + 0.01
    order = torch.randperm(T, generator=g, device="cuda")
    side = torch.where(order < int(math.floor(shift_frac * T + 0.5)), 1.0, -1.0)
    return torch.stack((-side * margin / 2, side * margin / 2), dim=1).contiguous()


def _weights(g, n, k, prepared):
    w = _w4(g, n, k)
    return sa.sa_shift_planes_prepare(w) if prepared else w


def _mlp(g, E, hid, moe, prepared, attn_std):
    """Weights and static scales of the MLP, by the rules of the repository's workloads."""
    y1_std = (127.0 / 4.0) * wl._RMS_W * math.sqrt(E)
    y2_std = 0.6 * wl._HIDDEN_UNITS_PER_ONE * wl._RMS_W * math.sqrt(hid)
    kw = dict(w1=_weights(g, hid, E, prepared), w2=_weights(g, E, hid, prepared),
              lut=torch.from_numpy(wl.activation_lut()).cuda(), act_inv_scale=127.0 / (4.0 * attn_std),
              requant_scale=wl._HIDDEN_UNITS_PER_ONE / y1_std, out_scale=1.0 / y2_std)
    if moe:
        kw["mw1"] = _randn(g, hid, E, std=1.0 / math.sqrt(E), dtype=torch.float16)
        kw["mw2"] = _randn(g, E, hid, std=1.0 / math.sqrt(hid), dtype=torch.float16)
    return kw


def _attention(case, N, nbits):
    """Mode, output scale and the rough standard deviation of the output (it sets the static int8 clip)."""
    if case["attention"] == "linear":
        return 0, 1.0 / math.sqrt(N * nbits), 1.0
    return 1, 1.0 / math.sqrt(nbits), 0.125


def _prepare_block(case, g):
    B, N, H, d, nbits, hid, moe = (case[k] for k in ("B", "N", "H", "d", "nbits", "hid", "moe"))
    mode, scale, std = _attention(case, N, nbits)
    kw = dict(B=B, N=N, H=H, d=d, nbits=nbits, dv=d, attention=mode, hid=hid, moe=moe, attn_scale=scale,
              q=_randn(g, B, N, H, d), k=_randn(g, B, N, H, d), v=_randn(g, B, N, H, d), proj=_randn(g, d, nbits),
              shift_variant=sa.SA_VARIANT_MFMA_PREPARED if case["prepared"] else sa.SA_VARIANT_AUTO)
    if hid:
        kw.update(_mlp(g, H * d, hid, moe, case["prepared"], std))
    if moe:
        kw["logits"] = _logits(g, B * N, case["shift_frac"])
    return sa.Block(**kw)


def _prepare_layer(case, g):
    B, N, H, E, nbits, hid, moe, prepared = (case[k] for k in ("B", "N", "H", "E", "nbits", "hid", "moe", "prepared"))
    mode, scale, std = _attention(case, N, nbits)
    T, acc_std = B * N, (127.0 / 4.0) * wl._RMS_W * math.sqrt(E)
    x = _randn(g, T, E)
    kw = dict(B=B, N=N, H=H, E=E, nbits=nbits, hid=hid, attention=mode, moe=moe, eps=1e-6, ln_inv_scale=127.0 / 4.0,
              qkv_scale=1.0 / acc_std, o_scale=1.0 / acc_std, attn_scale=scale,
              shift_variant=sa.SA_VARIANT_MFMA_PREPARED if prepared else sa.SA_VARIANT_AUTO,
              wqkv=_weights(g, 3 * E, E, prepared), wo=_weights(g, E, E, prepared),
              proj=None if case["sign_hash"] else _randn(g, E // H, nbits), **_mlp(g, E, hid, moe, prepared, std))
    for n in ("1", "2"):
        kw["gamma" + n] = 1.0 + _randn(g, E, std=0.1)
        kw["beta" + n] = _randn(g, E, std=0.1)
    if moe:
        # A trained router tells its tokens apart with a margin: the tokens carry a component along the direction the
        # router looks at, on the side of the expert they belong to.
        kw["wg"] = wg = _randn(g, E, 2, std=1.0 / math.sqrt(E))
        kw["bg"] = torch.zeros(2, device="cuda")
        u = wg[:, 1] - wg[:, 0]
        order = torch.randperm(T, generator=g, device="cuda")
        side = torch.where(order < int(math.floor(case["shift_frac"] * T + 0.5)), 1.0, -1.0)
        x += side[:, None] * (8.0 * u / u.norm())[None, :]
    return sa.Layer(x=x, **kw)


class _Conv01:
    """Hash, normalised linear attention on {0,1} codes, depthwise convolution of V added to it."""

    def __init__(self, case, g):
        B, gh, gw, H, d, nbits = (case[k] for k in ("B", "gh", "gw", "H", "d", "nbits"))
        N, E = gh * gw, H * d
        self.nbits, self.grid = nbits, (B, gh, gw, E)
        self.q, self.k, self.v = (_randn(g, B, N, H, d) for _ in range(3))
        self.proj, self.w, self.bias = _randn(g, d, nbits), _randn(g, E, 3, 3, std=1.0 / 3), _randn(g, E, std=0.1)
        self.codes = tuple(torch.empty((B, H, N, nbits // 64), dtype=torch.int64, device="cuda") for _ in range(2))
        self.kv = torch.empty((B, H, nbits, d), device="cuda")
        self.ksum = torch.empty((B, H, nbits), dtype=torch.int32, device="cuda")
        self.out = torch.empty((B, N, H, d), device="cuda")
        nbytes = sa.load_library().sa_linear_attention_01_workspace_bytes(B, H, N, N, nbits, d)
        self.ws = torch.empty(max(nbytes, 16), dtype=torch.uint8, device="cuda")

    def forward(self):
        qc, kc = sa.sa_binarize_pair(self.q, self.k, self.proj, self.nbits, *self.codes)
        sa.sa_linear_attention_01(qc, kc, self.v, 1e-6, self.nbits, kv=self.kv, ksum=self.ksum, out=self.out,
                                  workspace=self.ws)
        sa.sa_dwconv3x3(self.v.view(self.grid), self.w, self.bias, out=self.out.view(self.grid), accumulate=True)
        return {"codes": (qc, kc), "kv": self.kv, "ksum": self.ksum, "out": self.out}


class _Linears:
    """The two Shift layers of an MLP, int8 in, int32 out, on the packed weights."""

    def __init__(self, case, g):
        M, E, hid = case["M"], case["E"], case["hid"]
        self.x1, self.x2, self.w1, self.w2 = _int8(g, M, E), _int8(g, M, hid), _w4(g, hid, E), _w4(g, E, hid)
        self.bias = torch.randint(-5000, 5000, (hid,), generator=g, device="cuda", dtype=torch.int32)
        self.y1, self.y2 = (torch.empty((M, n), dtype=torch.int32, device="cuda") for n in (hid, E))
        nbytes = sa.sa_shift_planes_prepare(self.w1).numel() + 256
        self.ws = torch.empty(nbytes, dtype=torch.uint8, device="cuda")

    def forward(self):
        sa.sa_shift_linear(self.x1, self.w1, self.bias, y=self.y1, workspace=self.ws)
        sa.sa_shift_linear(self.x2, self.w2, y=self.y2, workspace=self.ws)
        return self.y1, self.y2


class _MoeLinear:
    def __init__(self, case, g):
        T, K, N = case["T"], case["K"], case["N"]
        x = _randn(g, T, K)
        self.xq, self.xh = sa.sa_quantize_act_half(x, 127.0 / 4.0)
        self.logits = _logits(g, T, case["shift_frac"])
        self.w4, self.wh = _w4(g, N, K), _randn(g, N, K, std=1.0 / math.sqrt(K), dtype=torch.float16)
        self.scale = 1.0 / ((127.0 / 4.0) * wl._RMS_W * math.sqrt(K))
        self.y = torch.empty((T, N), device="cuda")
        lib = sa.load_library()
        nbytes = lib.sa_moe_linear_workspace_bytes(sa._l(T), K, N, sa.SA_VARIANT_AUTO)
        self.ws = torch.empty(max(nbytes, 16), dtype=torch.uint8, device="cuda")

    def forward(self):
        return sa.sa_moe_linear(self.xq, self.xh, self.logits, self.w4, self.wh, self.scale, y=self.y, workspace=self.ws)


_PREPARE = {"block": _prepare_block, "layer": _prepare_layer, "conv01": _Conv01, "linears": _Linears,
            "moe_linear": _MoeLinear}


def prepare(case, seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed))
    return _PREPARE[case["kind"]](case, g)


def run(state):
    return state.forward()


# ------------------------------------------------------------------------- what a pass cannot do without --

def _attention_flops(B, N, H, nbits, dv, attention):
    if attention == "linear":
        return 4 * B * H * N * nbits * dv                    # K^T V and Q(K^T V)
    return 2 * B * H * N * N * dv                            # P V (the scores are integer compares of packed words)


def _mlp_work(T, E, hid, moe):
    """Weights read once (4 bits each, and fp16 for the Mult expert); either expert costs a token the same operations."""
    return E * hid + (4 * E * hid if moe else 0), 4 * T * E * hid


def work(case):
    kind = case["kind"]
    if kind == "block":
        B, N, H, d, nbits, hid, moe = (case[k] for k in ("B", "N", "H", "d", "nbits", "hid", "moe"))
        T, E = B * N, H * d
        nbytes, flops = 4 * 4 * T * E + 4 * d * nbits, 4 * T * H * d * nbits      # Q, K, V, O; the hash
        flops += _attention_flops(B, N, H, nbits, d, case["attention"])
        if hid:
            wb, wf = _mlp_work(T, E, hid, moe)
            nbytes, flops = nbytes + wb + 4 * T * E + (8 * T if moe else 0), flops + wf
    elif kind == "layer":
        B, N, H, E, nbits, hid, moe = (case[k] for k in ("B", "N", "H", "E", "nbits", "hid", "moe"))
        T, d = B * N, E // H
        wb, wf = _mlp_work(T, E, hid, moe)
        nbytes = 2 * 4 * T * E + 2 * E * E + wb               # tokens in and out, four attention Linears, the MLP
        flops = 8 * T * E * E + _attention_flops(B, N, H, nbits, d, case["attention"]) + wf
        if not case["sign_hash"]:
            flops += 4 * T * H * d * nbits
    elif kind == "conv01":
        B, N, H, d, nbits = case["B"], case["gh"] * case["gw"], case["H"], case["d"], case["nbits"]
        T, E = B * N, H * d
        nbytes = 4 * 4 * T * E + 2 * T * H * nbits // 8 + B * H * nbits * (d + 1) * 4
        flops = 4 * T * H * d * nbits + _attention_flops(B, N, H, nbits, d, "linear") + 18 * T * E
    elif kind == "linears":
        M, E, hid = case["M"], case["E"], case["hid"]
        nbytes, flops = 5 * M * (E + hid) + E * hid, 4 * M * E * hid
    else:
        T, K, N = case["T"], case["K"], case["N"]
        shift = int(math.floor(case["shift_frac"] * T + 0.5))
        nbytes = shift * K + 2 * (T - shift) * K + 8 * T + N * K // 2 + 2 * N * K + 4 * T * N
        flops = 2 * T * K * N
    return {"bytes": nbytes, "flops": flops}


def tolerance(case):
    if case["kind"] == "linears":
        return "exact"                                       # integers
    if case["kind"] == "layer" or (case["kind"] == "block" and case["hid"]):
        # An int8 quantiser stands between the float stages: a value that differs in its last bit can take the next code,
        # which moves its token's row by about 1e-2 of the rms.
        return {"rel": 5e-3, "max": 0.1}
    return {"rel": 1e-5, "max": 1e-3}                        # fp32 sums (of exact products, or of fp16 products)
