"""The split kernels' device functions (csrc/bhq_split.h), compiled for the
host with a stand-in for the HIP header, on inputs where they could go wrong."""
import ctypes
import importlib.util
import os
import re
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


def _functions(u):
    """erfc(u), g, G2, G3 and their logarithmic derivatives d ln F / d ln u."""
    c = 2.0 / np.sqrt(np.pi)
    w = c * u * np.exp(-u * u)
    ec = special.erfc(u)
    h = 2.0 * u * u * w
    k = 2.0 * u * u * h
    val = np.stack([ec, ec + w, 3.0 * (ec + w) + h, 15.0 * (ec + w) + 5.0 * h + k])
    # u d/du: erfc -> -w, w -> (1 - 2u^2) w, h -> (3 - 2u^2) h, k -> (5 - 2u^2) k
    dw, dh, dk = (1.0 - 2.0 * u * u) * w, (3.0 - 2.0 * u * u) * h, (5.0 - 2.0 * u * u) * k
    der = np.stack([-w, dw - w, 3.0 * (dw - w) + dh, 15.0 * (dw - w) + 5.0 * dh + dk])
    return val, der / val


def test_fp64_functions(host):
    """The FP64 radial functions over 0 < u < 4 at r_s = 1/2, where u and the
    table variable are exact, against 30 digits: no further off than the two
    polynomials of exp(-u^2) and erfcx (test_split_table.py) on the same points,
    in absolute and in relative r.m.s. and in the largest absolute error."""
    import mpmath as mp
    g = np.random.default_rng(6)
    u = np.concatenate([g.uniform(0.0, 4.0, 6000), np.arange(128) / 32.0,
                        np.nextafter(np.arange(1, 129) / 32.0, 0.0)])
    n = len(u)
    rs = np.full(n, 0.5)
    ref = []
    with mp.workdps(30):
        for v in u:
            v = mp.mpf(float(v))
            w = 2 / mp.sqrt(mp.pi) * v * mp.exp(-v * v)
            a, h = mp.erfc(v) + w, 2 * v * v * w
            ref.append((mp.erfc(v), a, 3 * a + h, 15 * a + 5 * h + 2 * v * v * h))
        P = ctypes.c_void_p
        stat = []
        for call in (host.split_functions_f64, host.split_functions_two_polynomials):
            out = np.zeros((n, 4))
            call(ctypes.c_int(n), P(u.ctypes.data), P(rs.ctypes.data), P(out.ctypes.data))
            err = np.array([[float(o - f) for o, f in zip(row, r)] for row, r in zip(out, ref)])
            rel = err / np.array(ref, float)
            stat.append((np.sqrt(np.mean(err ** 2, axis=0)), np.sqrt(np.mean(rel ** 2, axis=0)),
                         np.abs(err).max(axis=0)))
    for new, two in zip(*stat):
        assert np.all(new <= two), (new, two)


def test_fp64_table_matches_generator():
    spec = importlib.util.spec_from_file_location("gen64",
                                                  os.path.join(CSRC, "gen_split_table64.py"))
    gen = importlib.util.module_from_spec(spec)
    spec.loader.exec_module(gen)
    with open(os.path.join(CSRC, "split_erfc64.h")) as f:
        text = f.read()
    text = text[text.index("kErfc64["):]
    vals = [float(v) for v in re.findall(r"([-+0-9.]+e[-+0-9]+)", text[text.index("= {"):])]
    assert np.array_equal(np.array(vals).reshape(128, 10), np.array(gen.erfc_table()))


def test_fp32_functions(host):
    """The FP32 radial functions over 0 < u < 2.5 and r_s over three decades.
    The table variable is r times a rounded scale, rounded: each rounding has
    an r.m.s. of 0.42 units of 2^-24 (relative, over a decade of values), which
    a function takes up by its logarithmic derivative.  A function's own cubic
    adds its coefficients' and Horner's roundings, about 0.75 units together
    for one that is read off directly; composing the functions from each other
    takes several times that."""
    g = np.random.default_rng(5)
    n = 200000
    rs = 10.0 ** g.uniform(-3.0, 0.0, n)
    r = (g.uniform(0.0, 2.5, n) * 2.0 * rs * (1.0 - 1e-6)).astype(np.float32)
    out = np.zeros((n, 4), np.float32)
    P = ctypes.c_void_p
    host.split_functions_f32(ctypes.c_int(n), P(r.ctypes.data), P(rs.ctypes.data),
                             P(out.ctypes.data))
    val, der = _functions(r.astype(np.float64) / (2.0 * rs))
    unit = 2.0 ** -24
    for j, name in enumerate(("erfc", "g", "G2", "G3")):
        err = out[:, j] / val[j] - 1.0
        want = unit * np.sqrt(2.0 * 0.42 ** 2 * np.mean(der[j] ** 2) + 0.75 ** 2)
        rms = np.sqrt(np.mean(err ** 2))
        assert rms <= want, (name, rms, want)
        worst = unit * (2.0 * np.abs(der[j]) + 4.0)
        assert np.all(np.abs(err) <= worst), (name, np.abs(err / worst).max())
