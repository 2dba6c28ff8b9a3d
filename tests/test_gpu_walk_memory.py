"""GPU: device builds whose groups open more cells than the walk of the build
before was sized for, then as many, then few, on one context: the lists are
the host builder's bit for bit, and a rebuild of 131,072 particles at
theta = 0.2 (up to about 2000 cells opened) is walked level by level."""
import time

import pytest

from paper_1812_07313_amd import bhq, synth
from test_gpu_tree import _device, _host, _same

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def test_growing_walks():
    ctx = bhq.bhq_create(0, bhq.QUAD, bhq.FP32_OFS64)
    host = {}
    try:
        for k, (n, theta) in enumerate(((3000, 0.8), (3000, 0.0), (3000, 0.0), (5000, 0.0),
                                        (9000, 0.0), (9000, 0.0), (3000, 0.0), (3000, 0.0),
                                        (3000, 0.8), (9000, 0.3))):
            x, m = synth.plummer(n, synth.rng(49))
            h = host.setdefault((n, theta), _host(x, m, theta, 256, 1))
            _same(h, _device(ctx, x, m, theta, 256, 1), "build %d" % k)
    finally:
        bhq.bhq_destroy(ctx)


def test_rebuilds_keep_the_level_walk():
    """Rebuild at theta = 0.2 against theta = 0.4: 1.7 times as long, 12 times
    where the first build's overflow leaves the octet walk for good."""
    x, m = (torch.from_numpy(a).cuda() for a in synth.uniform_cube(131072, synth.rng(3)))
    t = []
    for theta in (0.4, 0.2):
        ctx = bhq.bhq_create(0, bhq.QUAD, bhq.FP32_OFS64)
        try:
            times = []
            for _ in range(6):
                torch.cuda.synchronize()
                t0 = time.perf_counter()
                bhq.bhq_build_lists_device(ctx, x, m, theta, 256)
                torch.cuda.synchronize()
                times.append(time.perf_counter() - t0)
            t.append(min(times))
        finally:
            bhq.bhq_destroy(ctx)
    assert t[1] < 5.0 * t[0], t
