"""Generate split_erfc64.h, the FP64 short-range kernels' table of erfc(u), and
split_table64.h, exp(-u^2) and the scaled complementary error function
erfcx(u) = exp(u^2) erfc(u), from which the kernels' table is checked when they
are compiled; all as piecewise polynomials.

The Gaussian-split radial functions (u = r / (2 r_s)) need E = exp(-u^2)
and erfc(u) = E erfcx(u).  Both are smooth; erfcx varies slowly (1 at
u = 0, about 1 / (sqrt(pi) u) for large u), and over an interval of width
h the logarithm of E changes by at most 2 u h.  On 0 <= u < U (U = 4:
cutoffs up to 8 r_s), cut into N = 64 intervals, a polynomial of degree 9
for E and one of degree 7 for erfcx per interval reach a few 1e-16
relative, evaluated by Horner's rule in FP64 (tests/test_split_table.py).
One index serves both:
    t = u N / U,  q = floor(t),  f = t - q in [0, 1),
    E(u) = e0 + f (e1 + ... + f e9),  erfcx(u) = x0 + f (x1 + ... + f x7).
Each polynomial interpolates its function at the Chebyshev points of the
interval (degree + 1 of them), computed with 50 significant digits (mpmath)
and rounded to FP64 once, coefficient by coefficient.  A row of the table
holds the interval's E coefficients followed by its erfcx coefficients.

The kernels need E only as the derivative of erfc (u = t / 32):
    erfc(u) = c0 + f (c1 + ... + f c9),  d erfc / dt = c1 + f (2 c2 + ... + 9 f^8 c9)
on 128 intervals of the same domain.  The derivative is the polynomial of degree
8 that interpolates it at the Chebyshev points of the interval, and c0 is erfc
at the interval's start; both are within 1e-19 of the functions before the
coefficients are rounded to FP64, once each.

    python paper_1812_07313_amd/csrc/gen_split_table64.py
"""
import os

import mpmath as mp

DOMAIN = 4
INTERVALS = 64
EXP_DEGREE = 9
ERFCX_DEGREE = 7
ERFC_INTERVALS = 128
ERFC_DEGREE = 9


def expm2(u):
    return mp.exp(-u * u)


def erfcx(u):
    return mp.exp(u * u) * mp.erfc(u)


def interval(fn, q, degree, domain=DOMAIN, n=INTERVALS):
    """Power-basis coefficients in f of fn on interval q (mpmath numbers)."""
    with mp.workdps(50):
        h = mp.mpf(domain) / n
        m = degree + 1
        fs = [(1 + mp.cos(mp.pi * (2 * j + 1) / (2 * m))) / 2 for j in range(m)]
        ys = [fn(q * h + h * f) for f in fs]
        V = mp.matrix([[f ** k for k in range(m)] for f in fs])
        c = mp.lu_solve(V, mp.matrix(ys))
        return [c[k] for k in range(m)]


def table(domain=DOMAIN, n=INTERVALS):
    """Rows [E c0..c9, erfcx c0..c7] per interval, rounded to FP64."""
    return [[float(v) for v in interval(expm2, q, EXP_DEGREE, domain, n)] +
            [float(v) for v in interval(erfcx, q, ERFCX_DEGREE, domain, n)]
            for q in range(n)]


def erfc_table(domain=DOMAIN, n=ERFC_INTERVALS):
    """Rows c0..c9 of erfc per interval, rounded to FP64."""
    rows = []
    with mp.workdps(50):
        h = mp.mpf(domain) / n
        for q in range(n):
            d = interval(lambda u: -2 * h / mp.sqrt(mp.pi) * expm2(u), q, ERFC_DEGREE - 1,
                         domain, n)
            rows.append([float(mp.erfc(q * h))] + [float(d[k] / (k + 1))
                                                   for k in range(ERFC_DEGREE)])
    return rows


def main():
    tab = table()
    stride = EXP_DEGREE + ERFCX_DEGREE + 2
    here = os.path.dirname(os.path.abspath(__file__))
    lines = [
        "// split_table64.h -- generated by gen_split_table64.py; do not edit.",
        "// exp(-u^2) and erfcx(u) = exp(u^2) erfc(u) on %d intervals of 0 <= u < %d:" % (
            INTERVALS, DOMAIN),
        "// row q = {degree-%d coefficients of exp(-u^2), degree-%d coefficients of" % (
            EXP_DEGREE, ERFCX_DEGREE),
        "// erfcx}, each in increasing powers of f = t - q, t = u %d / %d." % (INTERVALS, DOMAIN),
        "#pragma once",
        "",
        "namespace bhq {",
        "",
        "constexpr double kTab64Domain = %d.0;" % DOMAIN,
        "constexpr int kTab64Intervals = %d;" % INTERVALS,
        "constexpr int kExpDegree = %d;" % EXP_DEGREE,
        "constexpr int kErfcxDegree = %d;" % ERFCX_DEGREE,
        "constexpr int kTab64Stride = %d;  // kExpDegree + kErfcxDegree + 2" % stride,
        "constexpr double kTab64[kTab64Intervals][kTab64Stride] = {",
    ]
    for row in tab:
        lines.append("    {%s}," % ", ".join("%.17e" % v for v in row))
    lines += ["};", "", "}  // namespace bhq", ""]
    with open(os.path.join(here, "split_table64.h"), "w") as f:
        f.write("\n".join(lines))
    lines = [
        "// split_erfc64.h -- generated by gen_split_table64.py; do not edit.",
        "// erfc(u) on %d intervals of 0 <= u < %d: row q holds a polynomial's coefficients in" % (
            ERFC_INTERVALS, DOMAIN),
        "// increasing powers of f = t - q, t = u %d / %d, whose derivative is that of erfc too." % (
            ERFC_INTERVALS, DOMAIN),
        "#pragma once",
        "",
        "namespace bhq {",
        "",
        "constexpr double kErfcDomain = %d.0;" % DOMAIN,
        "constexpr int kErfcIntervals = %d;" % ERFC_INTERVALS,
        "constexpr int kErfcDegree = %d;" % ERFC_DEGREE,
        "constexpr int kErfcStride = kErfcDegree + 1;",
        "constexpr double kErfc64[kErfcIntervals][kErfcStride] = {",
    ]
    for row in erfc_table():
        lines.append("    {%s}," % ", ".join("%.17e" % v for v in row))
    lines += ["};", "", "}  // namespace bhq", ""]
    with open(os.path.join(here, "split_erfc64.h"), "w") as f:
        f.write("\n".join(lines))


if __name__ == "__main__":
    main()
