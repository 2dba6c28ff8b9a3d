"""The split kernels' device functions (csrc/bhq_split.h), compiled for the
host with a stand-in for the HIP header, on inputs where they could go wrong."""
import ctypes
import os
import subprocess

import numpy as np
import pytest
from scipy import special

from conftest import ROOT

HERE = os.path.join(ROOT, "tests")
CSRC = os.path.join(ROOT, "paper_1812_07313_amd", "csrc")


@pytest.fixture(scope="module")
def host(tmp_path_factory):
    so = str(tmp_path_factory.mktemp("split") / "split_host.so")
    subprocess.run(["g++", "-O2", "-std=gnu++17", "-ffp-contract=off", "-shared", "-fPIC",
                    "-I", os.path.join(HERE, "host_stub"), "-I", CSRC, "-o", so,
                    os.path.join(HERE, "split_host.cpp")], check=True)
    return ctypes.CDLL(so)


def _pairs(host, xi, xj, rs, rcut, cell):
    n = len(xi)
    a, kept = np.zeros((n, 4), np.float32), np.zeros(n, np.int32)
    P = ctypes.c_void_p
    host.split_pairs_f32(ctypes.c_int(n), P(xi.ctypes.data), P(xj.ctypes.data),
                         ctypes.c_double(rs), ctypes.c_double(rcut), ctypes.c_int(cell),
                         P(a.ctypes.data), P(kept.ctypes.data))
    return a, kept


@pytest.mark.parametrize("cell", [0, 1])
@pytest.mark.parametrize("reach", [1.0, 1e3, 2e4, 2e5])
def test_fp32_pairs_at_the_cutoff(host, cell, reach):
    """Pairs at r_cut = 5 r_s (the end of the FP32 table) whose i-particles lie
    `reach` cutoffs from the group's centre: their FP32 separation may exceed
    the cutoff by any amount where the FP64 decision keeps them, and must not
    lead out of the table.  The separations are along one axis, so that r has
    the error of two rounded offsets, together at most 2 reach 2^-24 of r_cut,
    and the force, which falls like exp(-u^2), is off by (2 u^2 + 3) times that,
    u = 2.5 (and the square of it)."""
    g = np.random.default_rng(3)
    n = 20000
    rcut = 9.91e-6  # 83.1 spacings of the FP32 offsets at the largest reach
    rs = rcut / 5.0
    xi = np.zeros((n, 3))
    xi[:, 0] = reach * rcut * g.uniform(0.6, 1.0, n)
    xj = xi.copy()
    xj[:, 0] += rcut * (1.0 - g.uniform(0.0, 1e-4, n))
    a, kept = _pairs(host, xi, xj, rs, rcut, cell)
    r = xj[:, 0] - xi[:, 0]
    assert np.array_equal(kept > 0, r * r < rcut * rcut)
    assert reach < 1e3 or np.count_nonzero(kept == 2) > 100
    a, r = a[kept > 0].astype(np.float64), r[kept > 0]
    assert np.all(np.isfinite(a))
    u = r / (2.0 * rs)
    ref = (special.erfc(u) + 2.0 / np.sqrt(np.pi) * u * np.exp(-u * u)) / r ** 2
    err = np.abs(a[:, 0] / ref - 1.0).max()
    d = (2.0 * 2.5 ** 2 + 3.0) * 2.0 * reach * 2.0 ** -24
    assert err <= d + d * d + 3e-6, err
