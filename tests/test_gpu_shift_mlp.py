"""Both layers of a Shift MLP in one launch: bit-identical to the two layers one after the other (integers up to the one
rounding of the output), and to the oracle, at every width and at the edges of its tiles, chunks and rules.  One launch leaves the
workspace's hidden rows alone, which says whether it ran."""
import numpy as np
import pytest
import torch

import oracle
from helpers import dev, host
from paper_2306_06446_amd import workloads as wl

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("rows,E,hid", [
    (1, 64, 256), (65, 64, 512), (3300, 64, 1536), (40000, 64, 384),            # 64 rows, two workgroups to a CU
    (1, 128, 256), (129, 128, 768), (16385, 128, 640),                          # 64 and 128 rows
    (63, 192, 384), (7681, 192, 768), (16400, 192, 256),
    (31, 256, 384), (10240, 256, 512), (16513, 256, 1024),
])
def test_one_launch_equals_the_two_layers(sa, rows, E, hid):
    g = torch.Generator(device="cuda")
    g.manual_seed(rows + E + hid)
    T = rows + 37
    xq = torch.randint(-127, 128, (T, E), generator=g, device="cuda", dtype=torch.int8)
    w1, w2 = (torch.randint(0, 256, s, generator=g, device="cuda", dtype=torch.uint8) for s in ((hid, E // 2), (E, hid // 2)))
    lut = torch.randint(-128, 128, (256,), generator=g, device="cuda", dtype=torch.int8)
    rq, out_scale = 127.0 / (4 * 40 * 73 * E ** 0.5), 1e-3
    perm = torch.randperm(T, generator=g, device="cuda").to(torch.int32)
    counts = torch.tensor([T - rows, rows], dtype=torch.int32, device="cuda")
    gate = torch.rand(T, generator=g, device="cuda")
    ws = torch.empty(T * hid + 4 * E * hid + 4096, dtype=torch.uint8, device="cuda")
    p1, p2 = sa.sa_shift_planes_prepare(w1), sa.sa_shift_planes_prepare(w2)
    old = torch.randn((T, E), generator=g, device="cuda")

    def go(stages, weights, variant, **kw):
        y = old.clone()
        for s in stages:
            sa.sa_shift_mlp(xq, *weights, rq, lut, want_y2=False, y=y, out_scale=out_scale, variant=variant, stages=s, workspace=ws, **kw)
        return y
    picked = dict(rows=perm, counts=counts, expert=1, max_rows=T, gate=gate)
    for flag in (0, 4):                                     # 4: SA_MLP_ACCUMULATE
        for kw in ({}, picked):
            ref = go((1, 2 | flag), (p1, p2), 3, **kw)
            assert torch.equal(go((3 | flag,), (p1, p2), 3, **kw), ref)
            assert torch.equal(go((3 | flag,), (w1, w2), 1, **kw), ref)
    n = min(rows, 96)                                       # the oracle on the last rows, ungated
    ref = oracle.shift_mlp(host(xq[-n:]), host(w1), host(w2), rq, host(lut))
    got = host(go((3,), (p1, p2), 3)[-n:])
    assert np.array_equal(got, np.float32(out_scale) * np.asarray(ref).astype(np.float32))


# either side of the sizes from which two launches are the faster way: the last round of one nearly empty, or nearly full
@pytest.mark.parametrize("rows,E,hid", [(16385, 256, 512), (21299, 256, 512), (32769, 256, 256), (32769, 192, 512), (45000, 192, 768),
                                        (32769, 128, 768), (46000, 128, 256)])
def test_the_last_round_of_rows(sa, rows, E, hid):
    test_one_launch_equals_the_two_layers(sa, rows, E, hid)


# One launch on decoded weights for certain: odd and even numbers of chunks of 128 hidden columns, 64 and 128 rows of a workgroup, all
# rows and a few that only the device counts.  Those keep two launches where one would be slower for some of the counts.
@pytest.mark.parametrize("T,E,hid,counted", [
    (3101, 192, 384, True), (16437, 192, 640, False), (7681, 192, 768, False), (4101, 256, 384, True), (17837, 256, 640, False),
    (22001, 256, 1024, False), (20001, 128, 384, True), (40001, 128, 640, True), (129, 128, 768, True), (12287, 128, 896, False),
    (12288, 128, 896, True), (16384, 192, 512, True), (16385, 192, 512, False), (11000, 256, 1024, False), (15000, 256, 2048, False),
    (11000, 192, 2048, False)])
def test_one_launch_it_is(sa, T, E, hid, counted):
    g = torch.Generator(device="cuda")
    g.manual_seed(T + E + hid)
    xq = torch.randint(-127, 128, (T, E), generator=g, device="cuda", dtype=torch.int8)
    w = [torch.randint(0, 256, s, generator=g, device="cuda", dtype=torch.uint8) for s in ((hid, E // 2), (E, hid // 2))]
    planes = [sa.sa_shift_planes_prepare(t) for t in w]
    lut = torch.randint(-128, 128, (256,), generator=g, device="cuda", dtype=torch.int8)
    rq = 127.0 / (4 * 40 * 73 * E ** 0.5)
    perm = torch.randperm(T, generator=g, device="cuda").to(torch.int32)
    gate = torch.rand(T, generator=g, device="cuda")
    ws = torch.zeros(T * hid + 4 * E * hid + 4096, dtype=torch.uint8, device="cuda")
    old = torch.randn((T, E), generator=g, device="cuda")

    def go(stages, **kw):
        y = old.clone()
        for s in stages:
            sa.sa_shift_mlp(xq, *planes, rq, lut, want_y2=False, y=y, out_scale=1e-3, variant=3, stages=s, workspace=ws, **kw)
        return y
    for kept in (None, 0, 1, 31, 65, T // 3, T):
        kw = {}
        if kept is not None:
            kw = dict(rows=perm, counts=torch.tensor([T - kept, kept], dtype=torch.int32, device="cuda"), expert=1, max_rows=T, gate=gate)
        ws.fill_(77)
        got = go((3,), **kw)
        untouched = bool((ws[:T * hid] == 77).all())
        assert kept == 0 or untouched == (counted or kept is None)
        ref = go((1, 2), **kw)
        assert torch.equal(got, ref)
        assert kept == 0 or not bool((ws[:T * hid] == 77).all())
        if kept is not None:
            idle = perm[:T - kept].long()
            assert torch.equal(got[idle], old[idle])


@pytest.mark.parametrize("T,E,hid", [(10999, 256, 1024), (14999, 256, 2048), (10999, 192, 2048), (8999, 128, 1536)])
def test_two_launches_they_are(sa, T, E, hid):
    test_one_launch_equals_the_two_layers(sa, T - 37, E, hid)
    g = torch.Generator(device="cuda")
    g.manual_seed(T)
    xq = torch.randint(-127, 128, (T, E), generator=g, device="cuda", dtype=torch.int8)
    w = [sa.sa_shift_planes_prepare(torch.randint(0, 256, s, generator=g, device="cuda", dtype=torch.uint8)) for s in ((hid, E // 2), (E, hid // 2))]
    ws = torch.full((T * hid + 4 * E * hid + 4096,), 77, dtype=torch.uint8, device="cuda")
    lut = torch.zeros(256, dtype=torch.int8, device="cuda")
    sa.sa_shift_mlp(xq, *w, 1e-3, lut, want_y2=False, y=torch.empty((T, E), device="cuda"), variant=3, workspace=ws)
    assert not bool(ws[:T * hid].any())                      # the hidden rows, all of them 0


# A tile of 128 rows for every CU, and one row more: the last rows whose workgroups take one tile each, and the first whose take several; hidden
# layers that are too long for that.
@pytest.mark.parametrize("rows,E,hid", [(32768 - 37, 128, 256), (32769 - 37, 128, 384), (32768 - 37, 192, 384), (32768 - 37, 256, 1024),
                                        (65536 - 37, 256, 640), (65536 - 37, 192, 512), (65536 - 37, 128, 1152)])
def test_a_tile_for_every_cu(sa, rows, E, hid):
    test_one_launch_equals_the_two_layers(sa, rows, E, hid)


# More than 256 tiles of 128 rows: a workgroup takes several, whole ones and the last one in part; two and three chunks of hidden columns,
# so that a ring of three stages comes round differently from tile to tile.
@pytest.mark.parametrize("rows,E,hid", [(65401, 256, 256), (65536, 256, 384), (90003, 192, 384), (65409, 128, 256), (98177, 128, 384)])
def test_tiles_one_after_the_other(sa, rows, E, hid):
    g = torch.Generator(device="cuda")
    g.manual_seed(rows + E + hid)
    T = rows + 131
    xq = torch.randint(-127, 128, (T, E), generator=g, device="cuda", dtype=torch.int8)
    w = [sa.sa_shift_planes_prepare(torch.randint(0, 256, s, generator=g, device="cuda", dtype=torch.uint8)) for s in ((hid, E // 2), (E, hid // 2))]
    lut = torch.randint(-128, 128, (256,), generator=g, device="cuda", dtype=torch.int8)
    rq = 127.0 / (4 * 40 * 73 * E ** 0.5)
    perm = torch.randperm(T, generator=g, device="cuda").to(torch.int32)
    gate, old = torch.rand(T, generator=g, device="cuda"), torch.randn((T, E), generator=g, device="cuda")
    ws = torch.empty(T * hid + 4 * E * hid + 4096, dtype=torch.uint8, device="cuda")

    def go(x, stages, **kw):
        y = old.clone()
        for s in stages:
            sa.sa_shift_mlp(x, *w, rq, lut, want_y2=False, y=y, out_scale=1e-3, variant=3, stages=s, workspace=ws, **kw)
        return y
    for flag in (0, 4):                                     # 4: SA_MLP_ACCUMULATE
        for x, kw in ((xq[:rows], {}), (xq, dict(rows=perm, max_rows=rows, gate=gate))):
            ws.fill_(77)
            got = go(x, (3 | flag,), **kw)
            assert bool((ws[:rows * hid] == 77).all())      # one launch
            assert torch.equal(got, go(x, (1, 2 | flag), **kw))
