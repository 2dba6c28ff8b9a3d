"""FP32 split kernels at r_cut = 5 r_s, the end of their table, with i-particles
2e5 cutoffs from their group's centre: a pair that the FP64 decision keeps may
have an FP32 separation well past the cutoff, where the table has no entries.

Tolerance as in test_split_host.py: r has the error of two rounded offsets, at
most 2 reach 2^-24 of r_cut = 2.4 %, which the force, falling like exp(-u^2),
takes up (2 u^2 + 3) = 15.5-fold (and its square); a missing or foreign table
entry gives another order of magnitude."""
import numpy as np
import pytest
from scipy import special

from paper_1812_07313_amd import bhq

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kernel", [bhq.SPLIT_MONO, bhq.SPLIT_QUAD])
@pytest.mark.parametrize("cells", [False, True])
def test_pairs_far_from_the_centre(kernel, cells):
    g = np.random.default_rng(3)
    n, reach, rs = 600, 2e5, 1.982e-6
    rcut = 5.0 * rs
    x = np.zeros((n, 3))
    x[:, 0] = reach * rcut * g.uniform(0.6, 1.0, n)
    x[:, 1] = np.arange(n) / 1024.0  # exact in FP32, pairs far apart
    xj = x.copy()
    xj[:, 0] += rcut * (1.0 - g.uniform(0.0, 1e-4, n))
    r = xj[:, 0] - x[:, 0]
    assert np.all(r * r < rcut * rcut)
    off, none = np.array([0, n], np.int64), np.array([0, 0], np.int64)
    ctx = bhq.bhq_create(0, kernel, bhq.FP32_OFS64)
    try:
        bhq.bhq_set_groups(ctx, off, np.zeros((1, 3)), none if cells else off,
                           off if cells else none)
        bhq.bhq_set_i(ctx, x)
        bhq.bhq_set_split(ctx, rs, rcut, 0.0)
        if cells:
            bhq.bhq_set_jc(ctx, 0, xj, np.ones(n), np.zeros((n, 6)), np.zeros(n))
        else:
            bhq.bhq_set_jp(ctx, 0, xj, np.ones(n))
        bhq.bhq_compute(ctx)
        a, _ = bhq.bhq_get_result(ctx, n)
    finally:
        bhq.bhq_destroy(ctx)
    u = r / (2.0 * rs)
    ref = (special.erfc(u) + 2.0 / np.sqrt(np.pi) * u * np.exp(-u * u)) / r ** 2
    d = (2.0 * 2.5 ** 2 + 3.0) * 2.0 * reach * 2.0 ** -24
    assert np.abs(a[:, 0] / ref - 1.0).max() <= d + d * d
    assert np.all(a[:, 1:] == 0.0)
