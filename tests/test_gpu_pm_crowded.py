"""GPU: the particle mesh with concentrated particles: mesh points whose cells
hold more particles than a block of the assignment goes over by itself (24),
against the FP64 particle-mesh reference, and the time they take."""
import numpy as np
import pytest

from oracle import pm as opm
from paper_1812_07313_amd import bhq, synth
from test_gpu_pm import _rel, _t

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def _cells(nmesh, counts, g):
    """Positions with counts[k] particles in the k-th of some cells, which
    include the box's faces and corner (a cell is the points nearest to a mesh
    point), and a few particles elsewhere."""
    cells = [(0, 0, 0), (nmesh - 1, 0, nmesh // 2), (nmesh // 2,) * 3,
             (1, nmesh - 1, nmesh - 1), (nmesh // 2, nmesh // 2, nmesh - 1)]
    x = [g.random((40, 3))]
    for c, k in zip(cells, counts):
        x.append(((np.array(c) + g.uniform(-0.49, 0.49, (k, 3))) / nmesh) % 1.0)
    return np.concatenate(x)


@pytest.mark.parametrize("nmesh", [4, 6, 16, 18, 34, 66])
@pytest.mark.parametrize("counts", [
    (24, 24, 24, 24, 24), (25, 0, 0, 0, 0),       # the last cell that a block takes, the next
    (0, 0, 25, 63, 64), (65, 500, 24, 1, 2000),   # edges of a wave's share
])
def test_crowded_cells(nmesh, counts):
    g = np.random.default_rng(nmesh + sum(counts))
    x = _cells(nmesh, counts, g)
    n = len(x)
    m = g.uniform(0.5, 1.5, n) / n
    rs = 1.25 / nmesh
    a_ref, p_ref = opm.pm(x, m, 1.0, nmesh, rs)
    pm = bhq.bhq_pm_create(nmesh, 1.0, rs)
    try:
        xt, mt = _t(x), _t(m)
        a = torch.full((n, 3), float("nan"), dtype=torch.float64, device="cuda")
        p = torch.full((n,), float("nan"), dtype=torch.float64, device="cuda")
        # twice, with a spread-out input between: the list of crowded blocks
        # is this evaluation's
        first = None
        for _ in range(2):
            bhq.bhq_pm_compute(pm, xt, mt, a, p)
            assert _rel(a.cpu().numpy(), a_ref) < 1e-11 and _rel(p.cpu().numpy(), p_ref) < 1e-11
            first = a.clone() if first is None else first
            assert torch.equal(a, first)
            bhq.bhq_pm_compute(pm, _t(g.random((n, 3))), mt, a, p)
    finally:
        bhq.bhq_pm_destroy(pm)


def test_concentrated_particles_take_little_longer():
    """A Plummer sphere of a twentieth of the box against as many particles
    spread evenly: 4 times as long (97 times where every block goes over its
    particles one by one)."""
    n, nmesh = 2000000, 128
    g = synth.rng(5)
    clump = (0.5 + 0.05 * synth.plummer(n, g)[0]) % 1.0
    m = _t(np.full(n, 1.0 / n))
    a = torch.zeros((n, 3), dtype=torch.float64, device="cuda")
    pm = bhq.bhq_pm_create(nmesh, 1.0, 1.25 / nmesh)
    try:
        ms = []
        for x in (g.random((n, 3)), clump):
            xt = _t(x)
            t = []
            for _ in range(4):
                bhq.bhq_pm_compute(pm, xt, m, a)
                t.append(bhq.bhq_pm_get_ms(pm))
            ms.append(min(t))
        assert ms[1] < 12.0 * ms[0], ms
    finally:
        bhq.bhq_pm_destroy(pm)
