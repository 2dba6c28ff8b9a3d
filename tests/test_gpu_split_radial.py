"""The FP64 split kernels' radial functions, one pair at a time: erfc(u) and
its derivative from one polynomial per interval of width 1/32 up to u = 4 and
from the library beyond.  Isolated pairs at separations u = r / 2 r_s on both
sides of interval ends, in their middles, close to zero and around u = 4, as
particle and as cell terms, against the FP64 oracle.

Tolerance: u carries about four roundings (r^2, its root, the scale), which the
functions, falling like exp(-u^2), amplify by up to 2 u^2 (41 at u = 4.5):
41 * 4 * 1.1e-16 = 1.8e-14, and as much again for the oracle's own u; with the
polynomials' and the products' few units below 4e-14."""
import numpy as np
import pytest

import oracle as orc
from _parity import run, upload
from paper_1812_07313_amd import bhq

pytestmark = pytest.mark.gpu

TOL = 4e-14


def _pairs(u, rs, seed):
    g = np.random.default_rng(seed)
    side = int(np.ceil(len(u) ** (1.0 / 3.0)))
    k = np.arange(len(u))
    c = (np.stack([k % side, (k // side) % side, k // side ** 2], axis=1) + 0.5) / side
    d = g.normal(size=(len(u), 3))
    d /= np.linalg.norm(d, axis=1)[:, None]
    x = np.empty((2 * len(u), 3))
    x[0::2] = c
    x[1::2] = c + (2.0 * rs * u)[:, None] * d
    return x, np.full(len(x), 1.0 / len(x))


@pytest.mark.parametrize("kernel", ["mono", "quad"])
def test_pairs_across_intervals(kernel):
    rs = 0.0015
    rcut = 9.0 * rs
    edges = np.arange(1, 129) / 32.0
    u = np.concatenate([[1e-3, 0.01], edges * (1.0 - 1e-12), edges * (1.0 + 1e-12),
                        edges - 1.0 / 64.0, [4.1, 4.3, 4.49]])
    x, m = _pairs(u, rs, 3)
    T = orc.Tree(x, m, 0.0, 2, nleaf=2, box=1.0, rcut=rcut)
    mat = orc.materialise(T, x, m)
    bk, ok = ((bhq.SPLIT_QUAD, orc.SPLIT_QUAD) if kernel == "quad"
              else (bhq.SPLIT_MONO, orc.SPLIT_MONO))
    a_ref, p_ref = orc.eval_lists(ok, mat, x, 0.0, box=1.0, rs=rs, rcut=rcut,
                                  mask=orc.MASK_F64_OFS)
    assert np.all(np.any(a_ref != 0.0, axis=1))
    ctx = bhq.bhq_create(0, bk, bhq.FP64)
    try:
        upload(ctx, mat, x, split=(rs, rcut, 1.0))
        a, p = run(ctx, mat, len(m), bk, bhq.FP64)
    finally:
        bhq.bhq_destroy(ctx)
    assert orc.relative_errors(a, a_ref).max() <= TOL
    assert (np.abs(p - p_ref) / np.abs(p_ref)).max() <= TOL
