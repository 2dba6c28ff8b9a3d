"""GPU: root cubes of a batch's systems where the width of their blocks changes
(a largest system of more than ten particles per system) and at the widths
themselves, bit for bit against the host builder's lists."""
import numpy as np
import pytest

from paper_1812_07313_amd import bhq, synth
from test_gpu_tree import _same

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("sizes", [
    (1,) * 29 + (300,), (1,) * 29 + (301,),
    (255, 256, 257, 1) * 8, (3,) * 200 + (1023, 1024, 1025, 2000), (1023, 1024, 1025),
])
def test_batch_roots(sizes):
    g = synth.rng(48)
    off = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int64)
    x = np.concatenate([synth.uniform_cube(k, g)[0] * g.uniform(0.1, 10.0) + g.normal(size=3)
                        for k in sizes])
    m = g.uniform(0.5, 1.5, len(x))
    L = bhq.bhq_build_lists_batch(off, x, m, 0.6, 16, 4)
    try:
        h = bhq.bhq_lists_export(L, len(m))
        h["cells"] = bhq.bhq_lists_cells(L)
        h["sizes"] = bhq.bhq_lists_sizes(L)
    finally:
        bhq.bhq_lists_free(L)
    ctx = bhq.bhq_create(0, bhq.QUAD, bhq.FP32_OFS64)
    try:
        bhq.bhq_build_lists_device_batch(ctx, off, torch.from_numpy(x).cuda(),
                                         torch.from_numpy(m).cuda(), 0.6, 16, 4)
        d = bhq.bhq_get_lists(ctx, len(m))
        d["cells"] = bhq.bhq_get_cells(ctx)
        d["sizes"] = bhq.bhq_get_lists_sizes(ctx)
        _same(h, d, "roots %d systems" % len(sizes))
    finally:
        bhq.bhq_destroy(ctx)
