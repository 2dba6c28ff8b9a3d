"""GPU: branches of the device list builder (bhq_build_lists_device) at the
sizes where they change, bit for bit against the host builder's lists."""
import numpy as np
import pytest

from paper_1812_07313_amd import bhq, synth
from test_gpu_tree import _device, _host, _same

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("n,theta,ncrit,nleaf", [
    (9, 0.5, 1, 1),          # a few cells
    (6000, 0.6, 64, 8),      # few groups: four waves walk each
    (9000, 0.6, 8, 4),       # more than 2048 groups: two waves each
    (5000, 0.0, 256, 1),     # groups that open more cells than a first build's LDS holds
    (9000, 0.0, 256, 1),     # ... than the walk's LDS can hold
])
def test_walk_branches(n, theta, ncrit, nleaf):
    """First build and rebuild (one walk into slots where the groups fit)."""
    x, m = synth.plummer(n, synth.rng(40))
    h = _host(x, m, theta, ncrit, nleaf)
    ctx = bhq.bhq_create(0, bhq.QUAD, bhq.FP32_OFS64)
    try:
        for build in range(3):
            _same(h, _device(ctx, x, m, theta, ncrit, nleaf), "walk %d build %d" % (n, build))
            longest = (int(np.diff(h["jp_off"]).max()), int(np.diff(h["jc_off"]).max()))
            assert bhq.bhq_get_build_info(ctx)[1:] == longest
    finally:
        bhq.bhq_destroy(ctx)


def _clumps(n, g):
    """Clumps of coincident and nearly coincident particles on a sphere."""
    x, m = synth.plummer(n, g)
    x[: n // 4] = x[0]
    x[n // 4: n // 2] = x[n // 4] + 1e-7 * g.random((n // 2 - n // 4, 3))
    return x, m


@pytest.mark.parametrize("n,ncrit,nleaf", [
    (1, 1, 1), (2, 1, 1),
    (254, 32, 8), (255, 32, 8), (256, 32, 8), (257, 33, 7),  # edges of a tile of particles
    (1022, 32, 8), (1023, 32, 8), (1024, 32, 8), (1025, 33, 7),
    (8192, 64, 8), (8193, 64, 8),
    (65536, 64, 8), (65537, 64, 8),    # one and four particles per thread
    (66559, 64, 8), (66560, 64, 8),    # edges of a tile of 1024
    (30000, 64, 8),                    # the scan of the tiles' counts in one block
    (800000, 256, 8),                  # ... and by several
    (9000, 4096, 1), (9000, 4097, 8),  # the longest group in windows, and past it
    (12000, 4097, 4097),               # leaves past it
])
def test_cells_from_keys(n, ncrit, nleaf):
    """Cells, groups, order and moments; a first build and a rebuild."""
    x, m = synth.plummer(n, synth.rng(41)) if n > 100000 else _clumps(n, synth.rng(41))
    h = _host(x, m, 0.8, ncrit, nleaf)
    ctx = bhq.bhq_create(0, bhq.QUAD, bhq.FP32_OFS64)
    try:
        for build in range(2):
            _same(h, _device(ctx, x, m, 0.8, ncrit, nleaf), "cells %d build %d" % (n, build))
    finally:
        bhq.bhq_destroy(ctx)


@pytest.mark.parametrize("n", [
    2047, 2048, 2049, 4096, 4097,      # one tile, two tiles and one merge
    16384, 16385,                      # eight tiles; seventeen of 1024 and two merges
    65535, 65536, 65537,               # eight runs of eight; tiles of 2048
    131072, 131073,                    # tiles of 4096
    262143, 262144, 262145,            # the largest; the library's sort
])
def test_sorted_tiles(n):
    """The order of the keys' sort: all bits on a first build, those of the
    last depth on a rebuild, with coincident particles (equal keys, which keep
    their input order) in different tiles."""
    g = synth.rng(42)
    x, m = synth.plummer(n, g)
    x[g.integers(0, n, 400)] = x[0]
    h = _host(x, m, 0.8, 256, 16)
    ctx = bhq.bhq_create(0, bhq.QUAD, bhq.FP32_OFS64)
    try:
        for build in range(2):
            _same(h, _device(ctx, x, m, 0.8, 256, 16), "tiles %d build %d" % (n, build))
    finally:
        bhq.bhq_destroy(ctx)


@pytest.mark.parametrize("sizes", [
    (1, 1, 3), (1023, 1, 1024, 5, 2000), (700,) * 9,
    tuple(range(1, 80)),               # many systems in one tile
])
@pytest.mark.parametrize("ncrit,nleaf", [(16, 4), (5000, 8)])
def test_batch_cells_from_keys(sizes, ncrit, nleaf):
    """Systems whose particles begin and end inside tiles, one of them of
    clumps; a first build (sorted as segments) and rebuilds (sorted in one go;
    the last deeper than the one before)."""
    g = synth.rng(42)
    off = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int64)
    shallow = [synth.uniform_cube(k, g) for k in sizes]
    deep = list(shallow)
    deep[-1] = _clumps(sizes[-1], g)
    ctx = bhq.bhq_create(0, bhq.QUAD, bhq.FP32_OFS64)
    try:
        for build, parts in enumerate((shallow, shallow, deep, deep)):
            x = np.concatenate([p[0] for p in parts])
            m = np.concatenate([p[1] for p in parts])
            L = bhq.bhq_build_lists_batch(off, x, m, 0.6, ncrit, nleaf)
            try:
                h = bhq.bhq_lists_export(L, len(m))
                h["cells"] = bhq.bhq_lists_cells(L)
                h["sizes"] = bhq.bhq_lists_sizes(L)
            finally:
                bhq.bhq_lists_free(L)
            bhq.bhq_build_lists_device_batch(ctx, off, torch.from_numpy(x).cuda(),
                                             torch.from_numpy(m).cuda(), 0.6, ncrit, nleaf)
            d = bhq.bhq_get_lists(ctx, len(m))
            d["cells"] = bhq.bhq_get_cells(ctx)
            d["sizes"] = bhq.bhq_get_lists_sizes(ctx)
            _same(h, d, "batch %d systems build %d" % (len(sizes), build))
    finally:
        bhq.bhq_destroy(ctx)


@pytest.mark.parametrize("ng", [1, 9, 2047, 2048, 2049, 9001])
@pytest.mark.parametrize("window,tail", [(256, 1024), (1024, 0), (1, 1)])
@pytest.mark.parametrize("skew", [False, True])
def test_order_plan(ng, window, tail, skew):
    """Edges of a tile of groups and of windows; skew: one group of nearly all
    the cost, so that the others share a piece longer than the table's first
    allocation; groups without i-particles cost nothing."""
    g = synth.rng(43)
    cnt = g.integers(0, 60, (3, ng))
    if skew:
        cnt[:, 0] = 100000
    off = [np.concatenate([[0], np.cumsum(c)]).astype(np.int64) for c in cnt]
    want = bhq.bhq_plan_order(off[0], off[1], off[2], window=window, tail=tail)
    ctx = bhq.bhq_create(0, bhq.QUAD, bhq.FP32_OFS64)
    try:
        bhq.bhq_set_group_order(ctx, bhq.ORDER_XCD, window, tail)
        t = [torch.from_numpy(o).cuda() for o in off]
        for _ in range(2):
            bhq.bhq_set_groups_dev(ctx, t[0], torch.zeros(ng, 3, dtype=torch.float64,
                                                          device="cuda"), t[1], t[2])
            assert np.array_equal(bhq.bhq_get_order(ctx), want)
    finally:
        bhq.bhq_destroy(ctx)


def test_upload_after_refusals():
    """Device set calls refused once, twice and three times in a row leave the
    context's arrays as they were, and the next good call is accepted (the
    check flags alternate between two words); parts of a list, with and
    without the trace; empty uploads."""
    g = synth.rng(44)
    n = 700  # entries of one group's lists, more than one block's elements
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a, np.float64)).cuda()  # noqa: E731
    x, m, q, tr = g.random((n, 3)), g.random(n), 0.1 * g.random((n, 6)), g.random(n)
    off = torch.tensor([0, n], dtype=torch.int64, device="cuda")

    def bad(a, k):
        b = np.array(a, np.float64)
        b.reshape(-1)[k] = np.inf
        return dev(b)

    def result(ctx):
        bhq.bhq_compute(ctx)
        return bhq.bhq_get_result(ctx, n)

    ctx = bhq.bhq_create(0, bhq.QUAD_SOFT, bhq.FP64)
    try:
        bhq.bhq_set_groups_dev(ctx, off, dev(np.full((1, 3), 0.5)), off, off)
        bhq.bhq_set_i_dev(ctx, dev(x))
        bhq.bhq_set_eps2_i_dev(ctx, dev(np.full(n, 1e-2)))
        bhq.bhq_set_jp_dev(ctx, 0, dev(x), dev(m))
        bhq.bhq_set_jc_dev(ctx, 0, dev(x[:400] + 2), dev(m[:400]), dev(q[:400]), dev(tr[:400]))
        bhq.bhq_set_jc_dev(ctx, 400, dev(x[400:] + 2), dev(m[400:]), dev(q[400:]))
        bhq.bhq_set_jp_dev(ctx, n, dev(x[:0]), dev(m[:0]))
        before = result(ctx)
        last = n - 1
        calls = (lambda: bhq.bhq_set_i_dev(ctx, bad(x, 3 * n - 1)),
                 lambda: bhq.bhq_set_eps2_i_dev(ctx, dev(np.arange(n) - 1.0)),
                 lambda: bhq.bhq_set_jp_dev(ctx, 0, dev(x + 1), bad(m, last)),
                 lambda: bhq.bhq_set_jc_dev(ctx, 0, dev(x), dev(m), bad(q, 6 * n - 1)),
                 lambda: bhq.bhq_set_jc_dev(ctx, 0, dev(x), dev(m), dev(q), bad(tr, last)))
        for times in (1, 2, 3):
            for call in calls:
                for _ in range(times):
                    with pytest.raises(bhq.BhqError) as e:
                        call()
                    assert e.value.code in (bhq.E_NONFINITE, bhq.E_ARG)
                after = result(ctx)
                assert np.array_equal(before[0], after[0]) and np.array_equal(before[1], after[1])
                bhq.bhq_set_i_dev(ctx, dev(x))
        # the kernels saw the trace where it was given and zero elsewhere
        bhq.bhq_set_jc_dev(ctx, 400, dev(x[400:] + 2), dev(m[400:]), dev(q[400:]),
                           dev(np.zeros(n - 400)))
        assert np.array_equal(before[0], result(ctx)[0])
        bhq.bhq_set_jc_dev(ctx, 0, dev(x[:400] + 2), dev(m[:400]), dev(q[:400]))
        assert not np.array_equal(before[0], result(ctx)[0])
        with pytest.raises(bhq.BhqError) as e:
            bhq.bhq_set_groups_dev(ctx, off, bad(np.zeros((1, 3)), 2), off, off)
        assert e.value.code == bhq.E_NONFINITE
        with pytest.raises(bhq.BhqError) as e:
            bhq.bhq_set_groups_dev(ctx, off, dev(np.zeros((1, 3))), off + 1, off)
        assert e.value.code == bhq.E_RANGE
        assert not np.array_equal(before[0], result(ctx)[0])  # still the lists above
    finally:
        bhq.bhq_destroy(ctx)


@pytest.mark.parametrize("kernel", [bhq.QUAD, bhq.MONO, bhq.QUAD_SOFT])
@pytest.mark.parametrize("dist,n,ncrit", [
    ("plummer", 60, 64),       # one group
    ("plummer", 2048, 64),     # few groups: parts
    ("plummer", 16384, 256),   # uneven groups: eight parts
    ("cube", 65536, 128),      # mean group sizes across the choices of
    ("cube", 30000, 128),      # i-particles per thread: 16, 58, 128
    ("cube", 524288, 256),
    ("cube", 24001, 512),      # blocks of 512: few large groups (375),
    ("plummer", 61003, 256),   # many of 64
])
def test_default_launch_shapes(kernel, dist, n, ncrit):
    """The launch shape that a context without bhq_set_tuning chooses, against
    the shape (256, 2) of one part in FP64; the same through
    bhq_compute_noalloc, after a rebuild, and on lists set from the host."""
    x, m = (synth.plummer if dist == "plummer" else synth.uniform_cube)(n, synth.rng(45))
    xt, mt = torch.from_numpy(x).cuda(), torch.from_numpy(m).cuda()
    ctx = bhq.bhq_create(0, kernel, bhq.FP64)
    try:
        bhq.bhq_set_eps(ctx, 0.01)
        bhq.bhq_set_tuning(ctx, 256, 2)
        bhq.bhq_build_lists_device(ctx, xt, mt, 0.7, ncrit)
        bhq.bhq_compute(ctx)
        ref = bhq.bhq_get_result(ctx, n)
    finally:
        bhq.bhq_destroy(ctx)
    for precision, rms, top in ((bhq.FP32_OFS64, 2e-6, 1e-4), (bhq.FP64, 1e-12, 1e-10)):
        ctx = bhq.bhq_create(0, kernel, precision)
        host = bhq.bhq_create(0, kernel, precision)
        try:
            shape = bhq.bhq_get_tuning(ctx)
            for c in (ctx, host):
                bhq.bhq_set_eps(c, 0.01)
            first = None
            for build in range(2):
                bhq.bhq_build_lists_device(ctx, xt, mt, 0.7, ncrit)
                bhq.bhq_compute(ctx)
                a, p = bhq.bhq_get_result(ctx, n)
                e = np.sqrt(((a - ref[0]) ** 2).sum(1) / (ref[0] ** 2).sum(1))
                assert np.sqrt(np.mean(e ** 2)) <= rms and e.max() <= top, (precision, e.max())
                assert (np.abs(p / ref[1] - 1)).max() <= top
                first = first or (a, p)
                assert np.array_equal(first[0], a) and np.array_equal(first[1], p)
            at = torch.empty(n, 3, dtype=torch.float64, device="cuda")
            pt = torch.empty(n, dtype=torch.float64, device="cuda")
            bhq.bhq_compute_noalloc(ctx, at, pt)
            assert np.array_equal(at.cpu().numpy(), a) and np.array_equal(pt.cpu().numpy(), p)
            L = bhq.bhq_build_lists(x, m, 0.7, ncrit)
            try:
                bhq.bhq_set_lists_indexed(host, L, x, m)
            finally:
                bhq.bhq_lists_free(L)
            bhq.bhq_set_eps(host, 0.01)
            bhq.bhq_compute(host)
            b, q = bhq.bhq_get_result(host, n)
            assert np.array_equal(a, b) and np.array_equal(p, q)
            assert bhq.bhq_get_tuning(ctx) == shape  # what the caller asked for
        finally:
            bhq.bhq_destroy(ctx)
            bhq.bhq_destroy(host)


def test_default_shape_captures():
    """A compute in parts that the context chose allocates nothing: it can be
    captured in a graph, whose replays give the eager result."""
    n = 4096
    x, m = synth.plummer(n, synth.rng(46))
    ctx = bhq.bhq_create(0, bhq.QUAD, bhq.FP32_OFS64)
    try:
        bhq.bhq_set_eps(ctx, 0.01)
        bhq.bhq_build_lists_device(ctx, torch.from_numpy(x).cuda(), torch.from_numpy(m).cuda(),
                                   0.6, 64)
        a = torch.zeros(n, 3, dtype=torch.float64, device="cuda")
        s = torch.cuda.Stream()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=s):
            bhq.bhq_compute_noalloc(ctx, a, None, stream=s)
        bhq.bhq_compute(ctx)
        want, _ = bhq.bhq_get_result(ctx, n)
        for _ in range(3):
            a.zero_()
            torch.cuda.synchronize()
            graph.replay()
            torch.cuda.synchronize()
            assert np.array_equal(a.cpu().numpy(), want)
            bhq.bhq_compute(ctx)
    finally:
        torch.cuda.synchronize()
        bhq.bhq_destroy(ctx)
