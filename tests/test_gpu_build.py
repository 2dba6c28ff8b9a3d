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
