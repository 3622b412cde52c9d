"""The MLP half of a layer and the MLP of a block in one launch for few rows, against the launches of their own that the same call makes
where the workspace has no room for that one: the same integer sums, the same order of the row's sums and, where those take the tiles that
split the contraction between four wavefronts, of the Mult expert's, so the same bits."""
import ctypes

import pytest
import torch

pytestmark = pytest.mark.gpu

RELU = torch.arange(-128, 128).clamp(min=0).to(torch.int8)


def rand(g, *shape):
    return torch.randn(shape, generator=g, device="cuda")


def weights(sa, g, E, hid, prepared, moe):
    w = {n: torch.randint(0, 256, s, generator=g, device="cuda", dtype=torch.uint8)
         for n, s in (("wqkv", (3 * E, E // 2)), ("wo", (E, E // 2)), ("w1", (hid, E // 2)), ("w2", (E, hid // 2)))}
    if prepared:
        w = {n: sa.sa_shift_planes_prepare(t) for n, t in w.items()}
    if moe:
        w.update(mw1=rand(g, hid, E).half() * E**-0.5, mw2=rand(g, E, hid).half() * hid**-0.5)
    return w


def layer(sa, T, E, ratio, moe, prepared=True, seed=0, bias=0.0, d=None, attention=0, nbits=64):
    """nbits = 0: the sign hash."""
    d = d or (64 if E != 64 else 32)
    g = torch.Generator(device="cuda")
    g.manual_seed(T + E + seed)
    hid = ratio * E
    x = rand(g, T, E)
    if T > 2:
        x[T // 2] = float("nan")
    kw = weights(sa, g, E, hid, prepared, moe)
    if moe:
        kw.update(wg=rand(g, E, 2) * E**-0.5, bg=torch.tensor([0.0, bias], device="cuda"))
    return sa.binding.Layer(B=1, N=T, H=E // d, nbits=nbits or d, E=E, hid=hid, attention=attention, moe=int(moe), shift_variant=3 if prepared else 2,
                            eps=1e-6, ln_inv_scale=32.0, qkv_scale=2.0**-12, attn_scale=(64.0 * T) ** -0.5, act_inv_scale=32.0,
                            o_scale=2.0**-12, requant_scale=2.0**-11, out_scale=2.0**-12, x=x, gamma1=1.0 + 0.1 * rand(g, E), beta1=0.1 * rand(g, E),
                            gamma2=1.0 + 0.1 * rand(g, E), beta2=0.1 * rand(g, E), proj=rand(g, d, nbits) if nbits else None,
                            lut=RELU.cuda(), **kw)


def block(sa, T, E, ratio, moe, prepared=True, seed=0, bias=0.0, d=None, attention=0, nbits=64):
    d = d or 32
    g = torch.Generator(device="cuda")
    g.manual_seed(T + E + seed)
    hid, H = ratio * E, E // d
    kw = weights(sa, g, E, hid, prepared, moe)
    del kw["wqkv"], kw["wo"]
    if moe:
        kw["logits"] = rand(g, T, 2) + torch.tensor([0.0, bias], device="cuda")
        kw["logits"][::5, 1] = kw["logits"][::5, 0]              # ties
    return sa.binding.Block(B=1, N=T, H=H, d=d, nbits=nbits or d, dv=d, attention=attention, hid=hid, moe=int(moe), attn_scale=(64.0 * T) ** -0.5,
                            act_inv_scale=32.0, requant_scale=2.0**-11, out_scale=2.0**-12, q=rand(g, 1, T, H, d), k=rand(g, 1, T, H, d),
                            v=rand(g, 1, T, H, d), proj=rand(g, d, nbits) if nbits else None, lut=RELU.cuda(), shift_variant=3 if prepared else 2, **kw)


def passes(made, n=1):
    out = []
    for _ in range(n):
        made.y.fill_(7.0)
        made.forward()
        out.append(made.y.clone().nan_to_num(nan=3.0))
    return out


def same(sa, made, n=2):
    got = passes(made, n)
    made.desc.workspace_bytes -= 1                               # launches of their own
    want, = passes(made)
    made.desc.workspace_bytes += 1
    assert float(want.abs().max()) > 0.0
    for y in got:
        assert torch.equal(y, want)


# one row, either side of a workgroup's 16, the last row count that takes 16, 32 and 64 of them
@pytest.mark.parametrize("moe", [True, False])
@pytest.mark.parametrize("T,E,ratio", [(1, 64, 8), (15, 128, 4), (16, 192, 4), (17, 256, 4), (33, 64, 4), (31, 128, 8), (50, 256, 8), (197, 192, 4),
                                       (512, 192, 4), (513, 192, 4), (512, 256, 4), (513, 256, 4), (1024, 192, 4), (1025, 192, 4),
                                       (1024, 256, 4), (2048, 192, 4), (1600, 64, 8), (1280, 128, 4)])
def test_layer_against_launches_of_their_own(sa, T, E, ratio, moe):
    same(sa, layer(sa, T, E, ratio, moe))


@pytest.mark.parametrize("T,E,ratio,moe", [(1, 192, 4, True), (1, 192, 4, False), (15, 64, 8, True), (16, 128, 4, False), (17, 192, 4, True),
                                           (17, 192, 4, False), (33, 256, 4, True), (416, 256, 4, True), (512, 192, 4, True), (1024, 192, 4, False),
                                           (1024, 128, 8, True), (1600, 128, 4, False), (1600, 64, 8, True), (1600, 64, 8, False),
                                           (112, 256, 8, True)])
def test_block_against_launches_of_their_own(sa, T, E, ratio, moe):
    same(sa, block(sa, T, E, ratio, moe))


# packed weights (Wo decoded with the MLP's); all rows with one expert, which leaves the other's workgroups none
@pytest.mark.parametrize("bias", [-100.0, 0.0, 100.0])
@pytest.mark.parametrize("prepared", [True, False])
@pytest.mark.parametrize("make", [layer, block])
def test_packed_weights_and_one_sided_routings(sa, make, prepared, bias):
    for T, E in ((49, 256), (197, 192), (500, 128)):
        same(sa, make(sa, T, E, 4, True, prepared, bias=bias))


# every kernel that clears what the launch counts with: the sign hash, alone or in the projection, and hashes of all code lengths, before either
# attention
@pytest.mark.parametrize("make", [layer, block])
@pytest.mark.parametrize("prepared", [True, False])
@pytest.mark.parametrize("attention", [0, 1])
@pytest.mark.parametrize("d,nbits", [(64, 0), (64, 64), (64, 128), (64, 256), (128, 0), (128, 128), (32, 64), (32, 128)])
def test_hashes_and_attentions(sa, make, prepared, attention, d, nbits):
    for T, E, moe in ((98, 128, True), (199, 256, True), (33, 64, False), (197, 192, True)):
        if E % d == 0:
            same(sa, make(sa, T, E, 4 if E > 64 else 8, moe, prepared, d=d, attention=attention, nbits=nbits))


def launches(made):
    """Nodes of the graph of one call."""
    passes(made)
    hip = ctypes.CDLL(next(l.split()[-1] for l in open("/proc/self/maps") if "libamdhip64" in l))
    graph = torch.cuda.CUDAGraph(keep_graph=True)
    with torch.cuda.graph(graph):
        made.forward()
    n = ctypes.c_size_t()
    assert hip.hipGraphGetNodes(ctypes.c_void_p(graph.raw_cuda_graph()), None, ctypes.byref(n)) == 0
    return n.value


# what the launch counts with is cleared by a launch that is there anyway
@pytest.mark.parametrize("nbits,most", [(0, 4), (64, 3)])        # the sign hash of Q and of K, or one hash for both; attention; MLP
@pytest.mark.parametrize("E,ratio,moe", [(64, 8, False), (128, 4, False), (192, 4, True)])
def test_no_launch_only_to_clear(sa, E, ratio, moe, nbits, most):
    assert launches(block(sa, 197, E, ratio, moe, d=64, nbits=nbits)) == most


@pytest.mark.parametrize("make", [layer, block])
def test_two_streams_and_replays(sa, make):
    """Two callers with workspaces of their own side by side; a captured call replayed between other work."""
    pair = [make(sa, 197, 192, 4, True, seed=s) for s in (1, 2)]
    want = [passes(m)[0] for m in pair]
    streams = [torch.cuda.Stream() for _ in pair]
    torch.cuda.synchronize()
    for _ in range(50):
        for m, st in zip(pair, streams):
            with torch.cuda.stream(st):
                m.forward()
    torch.cuda.synchronize()
    for m, y in zip(pair, want):
        assert torch.equal(m.y.clone().nan_to_num(nan=3.0), y)
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        pair[0].forward()
    for _ in range(4):
        pair[0].y.fill_(7.0)
        pair[0].ws.fill_(255)
        passes(pair[1])
        graph.replay()
        assert torch.equal(pair[0].y.clone().nan_to_num(nan=3.0), want[0])
