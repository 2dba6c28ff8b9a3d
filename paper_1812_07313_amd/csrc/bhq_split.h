// bhq_split.h -- the Gaussian-split (short-range) terms of the force kernels
// (device code): the tables of their radial functions, the functions, the
// cutoff decision, a particle and a cell term.  In a header of its own, so
// that tests can run these operations on the host as well.
#pragma once

#include <hip/hip_runtime.h>

#include <type_traits>

#include "bhq_terms.h"
#include "split_erfc64.h"
#include "split_table.h"
#include "split_table64.h"

namespace bhq {

__device__ __forceinline__ double erfc_r(double v) { return ::erfc(v); }
__device__ __forceinline__ double exp_r(double v) { return ::exp(v); }

// The FP64 kernels' table of erfc(u) (split_erfc64.h), copied to LDS by each
// block of an FP64 split kernel: on 128 intervals of 0 <= u < 4 a polynomial
// of degree 9 in f = t - q, t = 32 u, whose derivative gives exp(-u^2) as well.
// A pair then reads 80 B from LDS in place of the 144 of two polynomials
// (exp(-u^2) and erfcx); LDS bound the kernel (busy 66 % of the time and 15 %
// more in bank conflicts, VALU 72 %): the force kernel of a 60^3 lattice took
// 0.64 ms, then 0.56 (0.48 with far_g below).  The coefficients are rounded to FP64 once, from 50
// digits: against 64 bits and more the functions' r.m.s. errors (absolute,
// 1e-17, random r_s) are 2.9 (erfc), 5.3 (g), 7.5 / 3 (G2) and 8.9 / 15 (G3), those
// of the two polynomials 5.8, 7.5, 9.4 and 10.5; coefficients formed in FP64
// from the two polynomials gave 6.0, 8.1, 10.1 and 11.4.
struct Tab64 {
    double v[kErfcIntervals * kErfcStride];
};

constexpr Tab64 make_tab64()
{
    Tab64 t{};
    for (int q = 0; q < kErfcIntervals; ++q)
        for (int k = 0; k < kErfcStride; ++k) t.v[q * kErfcStride + k] = kErfc64[q][k];
    return t;
}

// The table agrees with exp(-u^2) and erfcx, interpolated by themselves
// (split_table64.h): erfc = exp(-u^2) erfcx and erfc' = -2/sqrt(pi) exp(-u^2) at
// the start and in the middle of their intervals.
constexpr bool erfc_table_agrees()
{
    constexpr double rsqpi2 = 1.12837916709551257389615890312;  // 2 / sqrt(pi)
    for (int q = 0; q < kErfcIntervals; ++q) {
        const double *c = kTab64[q / 2];
        const double f = 0.5 * (q % 2);
        double e = 0.0, x = 0.0;
        for (int k = kExpDegree; k >= 0; --k) e = e * f + c[k];
        for (int k = kErfcxDegree; k >= 0; --k) x = x * f + c[kExpDegree + 1 + k];
        const double v = kErfc64[q][0] / (e * x) - 1.0;
        const double d = kErfc64[q][1] * (kErfcIntervals / kErfcDomain) / (-rsqpi2 * e) - 1.0;
        if (!(v < 2e-15 && v > -2e-15 && d < 2e-15 && d > -2e-15)) return false;
    }
    return true;
}
static_assert(kErfcDomain == kTab64Domain && kErfcIntervals == 2 * kTab64Intervals &&
                  erfc_table_agrees(),
              "split_erfc64.h and split_table64.h: generate both again");

// The FP32 table of the split radial functions (split_table.h), one V4
// {c0, c1, c2, c3} per function and interval, likewise copied to LDS, where
// lanes read their own intervals.  One cubic of erfc on 641 intervals whose
// derivative gives the other functions reads half as much from LDS (a cell a
// quarter) and was 2 to 4 % faster, but its errors were larger: 1.1 (erfc) to
// 1.25 (G3) times these cubics' r.m.s. over random r_s.
struct SplitTab {
    V4<float> v[kSplitFuncs * kSplitEntries];
};

constexpr SplitTab make_split_tab()
{
    SplitTab t{};
    for (int f = 0; f < kSplitFuncs; ++f)
        for (int q = 0; q < kSplitEntries; ++q)
            t.v[f * kSplitEntries + q] = {kSplitTable[f][q][0], kSplitTable[f][q][1],
                                          kSplitTable[f][q][2], kSplitTable[f][q][3]};
    return t;
}

// Constants of the Gaussian split, uniform over a launch: u = r i2rs with
// i2rs = 1 / (2 r_s); the table variable is t = r ct = u N / U.
template <typename R>
struct SplitK {
    R i2rs;
    R ct;
};

template <typename R>
__device__ __forceinline__ SplitK<R> split_k(double rs)
{
    SplitK<R> K;
    const double i2rs = 0.5 / rs;
    K.i2rs = R(i2rs);
    K.ct = std::is_same<R, float>::value
               ? R(i2rs * (kSplitIntervals / (double)kSplitDomain))
               : R(i2rs * (kErfcIntervals / kErfcDomain));
    return K;
}

// Element type of the LDS table of a precision.
template <typename R>
struct SplitTabT {
    using type = V4<float>;
};
template <>
struct SplitTabT<double> {
    using type = double;
};
template <typename R>
using TabT = typename SplitTabT<R>::type;

// Gaussian-split radial functions at r (r2 = r^2), u = r / (2 r_s):
//   ec = erfc(u), g = erfc(u) + (2u/sqrt(pi)) e^{-u^2},
//   G2 = 3g + h, G3 = 15g + 5h + k, with h = (4u^3/sqrt(pi)) e^{-u^2} and
//   k = 2 u^2 h (G2, G3 only for cells with the quadrupole).
// FP64 takes erfc(u) and its derivative in t from one polynomial (interval
// q = floor(t), t = 32 u, f = t - q, Horner's rule for both): t times the
// derivative is u erfc'(u) = -(2u/sqrt(pi)) e^{-u^2}.  Past u = 4, that is for
// cutoffs beyond 8 r_s, it calls the library's exp and erfc.  FP32 reads the
// piecewise cubics of its table at t = r ct: interval q = floor(t), local
// variable f = t - q, Horner's rule (valid for u up to kSplitDomain and one
// interval beyond; the host refuses FP32 split kernels with a longer
// cutoff).
template <typename R>
struct SplitG {
    R ec, g, g2, g3;
};

__device__ __forceinline__ float horner(const V4<float> &c, float f)
{
    return fmaf(fmaf(fmaf(c.w, f, c.z), f, c.y), f, c.x);
}

// erfc(u) and e^{-u^2} past the FP64 table, from the library.  A function that
// is not inlined: inlined, its constants were kept over the loops of lists
// that never come here, in registers spilled to scratch memory by every block
// (252 bytes a lane), and each unrolled pair had its copy.  FP64 quadrupole
// kernel, ms, inlined / called: lattice 110^3 in 239,675 groups 10.5 / 4.5,
// 60^3 in 4096 groups 0.52 / 0.44; cutoff 12 r_s, 48^3, 1.6 / 0.62.
struct FarG {
    double ec, e;
};

__device__ inline __attribute__((noinline)) FarG far_g(double u)
{
    return {erfc_r(u), exp_r(-u * u)};
}

template <typename R, bool CELL>
__device__ __forceinline__ SplitG<R> split_g(R r, const SplitK<R> &K, const TabT<R> *tab)
{
    SplitG<R> s;
    if constexpr (std::is_same<R, float>::value) {
        const float t = r * K.ct;
        const int q = (int)t;  // t >= 0
        const float f = __builtin_amdgcn_fractf(t);
        s.ec = horner(tab[q], f);
        s.g = horner(tab[kSplitEntries + q], f);
        if (CELL) {
            s.g2 = horner(tab[2 * kSplitEntries + q], f);
            s.g3 = horner(tab[3 * kSplitEntries + q], f);
        }
    } else {
        const R t = r * K.ct;
        R w;  // (2u/sqrt(pi)) e^{-u^2} = -u erfc'(u)
        if (t < R(kErfcIntervals)) {
            const int q = (int)t;
            const R f = t - R(q);
            const double *c = tab + q * kErfcStride;
            R d = c[kErfcDegree];
            s.ec = fma(d, f, c[kErfcDegree - 1]);
#pragma unroll
            for (int k = kErfcDegree - 2; k >= 0; --k) {
                d = fma(d, f, s.ec);
                s.ec = fma(s.ec, f, c[k]);
            }
            w = -t * d;
            s.g = fma(-t, d, s.ec);
        } else {
            const R u = r * K.i2rs;
            const FarG far = far_g(u);
            s.ec = far.ec;
            w = R(1.12837916709551257389615890312) * u * far.e;
            s.g = s.ec + w;
        }
        if (CELL) {
            const R u = r * K.i2rs;
            const R u2 = R(2) * u * u;
            const R h = u2 * w;
            const R k = u2 * h;
            s.g2 = fma(R(3), s.g, h);
            s.g3 = fma(R(15), s.g, fma(R(5), h, k));
        }
    }
    return s;
}

// The cutoff is a decision on r^2, which the FP32 kernels form from FP32
// offsets.  It is taken as the FP64 kernel takes it: FP64 offsets
// X = wrap(v - c) from the group centre c, D = X_j - X_i, r^2 =
// fma(Dz, Dz, fma(Dy, Dy, Dx Dx)), kept iff 0 < r^2 < rcut * rcut in FP64.
// Outside a band around fl32(rcut^2) the FP32 r^2 decides the same way; a
// term inside the band (rare) is decided again from the FP64 positions.
//
// Band: with u = 2^-24, FP32 offsets x = X (1 + e), |e| <= u, the FP32
// difference and the three-term FMA chain give, to first order in u,
// |r2_32 - |D|^2| <= 7 u |D|^2 + 4 u |X_i| |D|, and fl32(rcut^2) is within
// u rcut^2 of rcut^2 (the FP64 side is exact to 2^-50).  Near the cutoff
// |D| ~ rcut, so u (8 rcut^2 + 4 |X_i| rcut) bounds the difference;
// band_i = u (16 rcut^2 + 8 |X_i| rcut) doubles it.  A term with
// |r2_32 - fl32(rcut^2)| >= band_i is on the same side in both precisions.
__device__ __forceinline__ float cut_band(float xi, float yi, float zi, float rcut)
{
    const float xn = __builtin_sqrtf(fmaf(zi, zi, fmaf(yi, yi, xi * xi)));
    return 0x1p-21f * rcut * fmaf(2.0f, rcut, xn);  // u (16 rcut^2 + 8 |X_i| rcut)
}

// FP64 cutoff decision of the FP64 kernel for the FP64 offsets xj - xi
// (each already wrapped relative to the group centre).
__device__ __forceinline__ bool keep_f64(double djx, double djy, double djz, double rcut)
{
    const double r2 = fma(djz, djz, fma(djy, djy, djx * djx));
    return r2 > 0.0 && r2 < rcut * rcut;
}

// Separation of a list entry from an i-particle and its squared length.
template <typename R>
struct Sep {
    R dx, dy, dz, r2;
};

template <typename R>
__device__ __forceinline__ Sep<R> separation(const V4<R> &j, R xi, R yi, R zi)
{
    Sep<R> s;
    s.dx = j.x - xi;
    s.dy = j.y - yi;
    s.dz = j.z - zi;
    s.r2 = fma(s.dz, s.dz, fma(s.dy, s.dy, s.dx * s.dx));
    return s;
}

// A separation that the FP64 decision kept: its FP32 r^2 may still exceed
// rcut^2 (by the rounding of the offsets, which is as large as the
// i-particle is far from the group's centre), and with r_cut at the end of the
// table's domain it would lead out of the table.
template <typename R>
__device__ __forceinline__ Sep<R> within_cutoff(Sep<R> s, R rcut2)
{
    s.r2 = s.r2 < rcut2 ? s.r2 : rcut2;
    return s;
}

// Short-range particle at separation s, kept by the cutoff decision:
// a += m g/r^3 d, -phi += m erfc(u)/r.
template <typename R>
__device__ __forceinline__ void pp_split(const V4<R> &j, const Sep<R> &s, const SplitK<R> &K,
                                         const TabT<R> *tab, R &ax, R &ay, R &az, R &pt)
{
    const R rinv = rsq(s.r2);
    const R r = s.r2 * rinv;
    const SplitG<R> f = split_g<R, false>(r, K, tab);
    const R mr = j.w * rinv;
    const R c = mr * f.g * (rinv * rinv);
    pt = fma(mr, f.ec, pt);
    ax = fma(c, s.dx, ax);
    ay = fma(c, s.dy, ay);
    az = fma(c, s.dz, az);
}

// Short-range cell expanded to second order about its centre of mass
// (with the trace T):
//   phi = M Phi + D2 dQd / 6 + T/6 (D2 r^2 + 3 D1)
//   a   = [M D1 + D3 dQd / 6 + T/6 (D3 r^2 + 5 D2)] d + D2/3 Qd
// with D1 = g/r^3, D2 = -(3g + h)/r^5, D3 = (15g + 5h + k)/r^7.
template <typename R, bool QUAD>
__device__ __forceinline__ void pc_split(const V4<R> &a, const V4<R> &b, const V4<R> &c,
                                         const Sep<R> &s, const SplitK<R> &K,
                                         const TabT<R> *tab, R &ax, R &ay, R &az, R &pt)
{
    const R dx = s.dx, dy = s.dy, dz = s.dz, r2 = s.r2;
    const R rinv = rsq(r2);
    const R r = r2 * rinv;
    const R rinv2 = rinv * rinv;
    const SplitG<R> f = split_g<R, QUAD>(r, K, tab);
    const R D1 = f.g * rinv2 * rinv;
    R phi = -a.w * f.ec * rinv;  // M Phi
    R coef = a.w * D1;
    if (QUAD) {
        const R rinv5 = rinv2 * rinv2 * rinv;
        const R D2 = -f.g2 * rinv5;
        const R D3 = f.g3 * rinv5 * rinv2;
        const R qx = fma(b.z, dz, fma(b.y, dy, b.x * dx));
        const R qy = fma(c.x, dz, fma(b.w, dy, b.y * dx));
        const R qz = fma(c.y, dz, fma(c.x, dy, b.z * dx));
        const R dqd = fma(dz, qz, fma(dy, qy, dx * qx));
        const R t6 = c.z * R(1.0 / 6.0);
        phi = fma(D2, dqd * R(1.0 / 6.0), phi);
        phi = fma(t6, fma(D2, r2, R(3) * D1), phi);
        coef = fma(D3, dqd * R(1.0 / 6.0), coef);
        coef = fma(t6, fma(D3, r2, R(5) * D2), coef);
        const R d23 = D2 * R(1.0 / 3.0);
        ax = fma(d23, qx, ax);
        ay = fma(d23, qy, ay);
        az = fma(d23, qz, az);
    }
    pt -= phi;
    ax = fma(coef, dx, ax);
    ay = fma(coef, dy, ay);
    az = fma(coef, dz, az);
}

}  // namespace bhq
