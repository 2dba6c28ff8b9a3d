"""GPU: the particle mesh at the sizes where its kernels' tiles begin and end,
against the FP64 particle-mesh reference."""
import numpy as np
import pytest

from oracle import pm as opm
from paper_1812_07313_amd import bhq
from test_gpu_pm import _rel, _t

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("nmesh,density", [
    (4, 3.0), (4, 0.05),              # smaller than a tile: cells met several times
    (6, 1.0), (14, 1.0),
    (16, 1.3), (18, 1.3), (32, 0.02),  # edges of a tile; long runs of empty cells
    (34, 4.0),                         # planes in several parts
    (50, 1.0), (66, 0.6),
])
@pytest.mark.parametrize("clumped", [False, True])
def test_pm_tiles(nmesh, density, clumped):
    n = max(1, int(density * nmesh ** 3))
    g = np.random.default_rng(nmesh)
    x = g.random((n, 3))
    if clumped:  # most particles in few cells, some on the faces of the box
        x[n // 3:] = (0.98 + 0.03 * x[n // 3:]) % 1.0
        x[: n // 10] = np.floor(x[: n // 10] * nmesh) / nmesh
    m = g.uniform(0.5, 1.5, n) / n
    rs = 1.25 / nmesh
    a_ref, p_ref = opm.pm(x, m, 1.0, nmesh, rs)
    pm = bhq.bhq_pm_create(nmesh, 1.0, rs)
    try:
        xt, mt = _t(x), _t(m)
        a = torch.full((n, 3), float("nan"), dtype=torch.float64, device="cuda")
        p = torch.full((n,), float("nan"), dtype=torch.float64, device="cuda")
        bhq.bhq_pm_compute(pm, xt, mt, a, p)
        a0, p0 = a.cpu().numpy(), p.cpu().numpy()
        assert _rel(a0, a_ref) < 1e-11 and _rel(p0, p_ref) < 1e-11
        # without the potential, added, and the same bits again
        b = torch.ones_like(a)
        bhq.bhq_pm_compute(pm, xt, mt, b, None, accumulate=True)
        assert np.array_equal(b.cpu().numpy(), 1.0 + a0)
    finally:
        bhq.bhq_pm_destroy(pm)


@pytest.mark.parametrize("nmesh", [128, 130])
def test_pm_batched_transforms(nmesh):
    """The largest mesh whose inverse transforms run as one batch, and the
    next."""
    n = 100000
    g = np.random.default_rng(nmesh)
    x, m = g.random((n, 3)), g.uniform(0.5, 1.5, n) / n
    rs = 1.25 / nmesh
    a_ref, p_ref = opm.pm(x, m, 1.0, nmesh, rs)
    pm = bhq.bhq_pm_create(nmesh, 1.0, rs)
    try:
        a = torch.zeros((n, 3), dtype=torch.float64, device="cuda")
        p = torch.zeros(n, dtype=torch.float64, device="cuda")
        bhq.bhq_pm_compute(pm, _t(x), _t(m), a, p)
        assert _rel(a.cpu().numpy(), a_ref) < 1e-11 and _rel(p.cpu().numpy(), p_ref) < 1e-11
    finally:
        bhq.bhq_pm_destroy(pm)
