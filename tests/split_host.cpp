// The split kernels' operations (csrc/bhq_split.h) compiled for the host, for
// test_split_host.py.
#include <cstring>
#include <limits>
#include <random>
#include <vector>

#include "bhq_split.h"

using namespace bhq;

namespace {

// An FP32 table as a block of a split kernel holds it, with NaN behind it.
const V4<float> *guarded_table()
{
    static std::vector<V4<float>> v;
    if (v.empty()) {
        static const SplitTab t = make_split_tab();
        const float nan = std::numeric_limits<float>::quiet_NaN();
        const size_t n = sizeof(t.v) / sizeof(t.v[0]);
        v.assign(t.v, t.v + n);
        v.resize(2 * n, V4<float>{nan, nan, nan, nan});
    }
    return v.data();
}

}  // namespace

extern "C" {

// erfc(u), g, G2, G3 (out[4k ..]) at r[k] with the split scale rs[k], as the
// FP32 kernels form them.
void split_functions_f32(int n, const float *r, const double *rs, float *out)
{
    for (int k = 0; k < n; ++k) {
        const SplitG<float> f = split_g<float, true>(r[k], split_k<float>(rs[k]),
                                                     guarded_table());
        const float o[4] = {f.ec, f.g, f.g2, f.g3};
        std::memcpy(out + 4 * k, o, sizeof(o));
    }
}

// The same of the FP64 kernels.
void split_functions_f64(int n, const double *r, const double *rs, double *out)
{
    static const Tab64 tab = make_tab64();
    for (int k = 0; k < n; ++k) {
        const SplitG<double> f = split_g<double, true>(r[k], split_k<double>(rs[k]), tab.v);
        const double o[4] = {f.ec, f.g, f.g2, f.g3};
        std::memcpy(out + 4 * k, o, sizeof(o));
    }
}

// The same from the two polynomials of split_table64.h (exp(-u^2) and erfcx).
void split_functions_two_polynomials(int n, const double *r, const double *rs, double *out)
{
    for (int k = 0; k < n; ++k) {
        const double u = r[k] * (0.5 / rs[k]), u2 = u * u;
        const double t = u * (kTab64Intervals / kTab64Domain);
        const int q = (int)t;
        const double f = t - q;
        const double *c = kTab64[q], *cx = c + kExpDegree + 1;
        double E = c[kExpDegree], x = cx[kErfcxDegree];
        for (int i = kExpDegree - 1; i >= 0; --i) E = fma(E, f, c[i]);
        for (int i = kErfcxDegree - 1; i >= 0; --i) x = fma(x, f, cx[i]);
        const double e = E * 0.56418958354775628694807945156;
        const double ec = E * x, g = fma(2 * u, e, ec), h = 4 * u * u2 * e;
        const double o[4] = {ec, g, fma(3.0, g, h), fma(15.0, g, fma(5.0, h, 2 * u2 * h))};
        std::memcpy(out + 4 * k, o, sizeof(o));
    }
}

// n pairs, offsets xi, xj (FP64, from the group centre): the FP32 split
// kernels' acceleration (a[4k .. 4k + 2]) and potential (negative, a[4k + 3])
// of a unit mass at xj on xi, as a particle (cell 0) or as a cell without
// moments (cell 1); kept[k]: 0 outside the cutoff, 1 inside, 2 inside by the
// FP64 decision.
void split_pairs_f32(int n, const double *xi, const double *xj, double rs, double rcut, int cell,
                     float *a, int *kept)
{
    const V4<float> *tab = guarded_table();
    const SplitK<float> K = split_k<float>(rs);
    const float rcut2 = (float)(rcut * rcut);
    for (int k = 0; k < n; ++k) {
        const double *p = xi + 3 * k, *q = xj + 3 * k;
        const V4<float> j = {(float)q[0], (float)q[1], (float)q[2], 1.0f};
        const float x = (float)p[0], y = (float)p[1], z = (float)p[2];
        const float band = cut_band(x, y, z, (float)rcut);
        Sep<float> s = separation(j, x, y, z);
        kept[k] = s.r2 > 0.0f && s.r2 < rcut2 - band ? 1 : 0;
        if (s.r2 >= rcut2 - band && s.r2 < rcut2 + band &&
            keep_f64(q[0] - p[0], q[1] - p[1], q[2] - p[2], rcut)) {
            s = within_cutoff(s, rcut2);
            kept[k] = 2;
        }
        float o[4] = {0.0f, 0.0f, 0.0f, 0.0f};
        if (kept[k] && cell) {
            const V4<float> zero = {0.0f, 0.0f, 0.0f, 0.0f};
            pc_split<float, true>(j, zero, zero, s, K, tab, o[0], o[1], o[2], o[3]);
        } else if (kept[k]) {
            pp_split(j, s, K, tab, o[0], o[1], o[2], o[3]);
        }
        std::memcpy(a + 4 * k, o, sizeof(o));
    }
}

}  // extern "C"
