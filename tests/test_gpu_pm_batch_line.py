"""GPU: the largest mesh whose inverse transforms run as one batch (224), and
the next, against the FP64 particle-mesh reference."""
import numpy as np
import pytest

from oracle import pm as opm
from paper_1812_07313_amd import bhq
from test_gpu_pm import _rel, _t

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("nmesh", [224, 226])
def test_pm_batch_line(nmesh):
    n = 20000
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
