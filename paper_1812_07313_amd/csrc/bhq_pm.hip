// bhq_pm.hip -- particle-mesh long-range force, the complement of the
// Gaussian-split short-range tree kernels (together: TreePM; the paper's
// TreePM context, Sec. 1).
//
// The short-range pair potential is -erfc(r / 2 r_s) / r, so the long-range
// part is -erf(r / 2 r_s) / r, whose Fourier transform is
// -4 pi exp(-k^2 r_s^2) / k^2.  In the periodic box of side L (mean density
// removed, G = 1) on an n^3 mesh of spacing h = L / n:
//   1. triangular-shaped-cloud (TSC) assignment of the masses (mesh points
//      at integer multiples of h): the particles are radix-sorted by their
//      nearest mesh point, and a thread per column of mesh points sums, in a
//      fixed order, the particles of the 27 cells around each (no atomics:
//      the result is the same bits every run); a wave per mesh point does so
//      around crowded cells;
//   2. forward real-to-complex FFT (hipFFT);
//   3. one thread per complex mode: phi(k) = G(k) rho(k) with
//      G = -4 pi exp(-k^2 r_s^2) / k^2 / W(k)^2, W = prod_a sinc(k_a h/2)^3
//      (TSC window, assignment and interpolation), G(0) = 0, and the three
//      components -i k_a phi(k) (zero on the Nyquist planes);
//   4. four inverse complex-to-real FFTs (acceleration and potential);
//   5. one thread per particle, in the sorted order, interpolates the four
//      meshes with the same TSC weights and writes its result at the
//      particle's input position.  A block takes the particles of a tile of
//      4 x 8 x 16 cells, with the fields at the tile's mesh points and their
//      neighbours in LDS.
// All FP64.
#include <hip/hip_runtime.h>
#include <hipcub/hipcub.hpp>
#include <hipfft/hipfft.h>

#include <cmath>
#include <cstdarg>
#include <cstdio>
#include <new>
#include <string>

#include "bhq.h"
#include "bhq_internal.h"
#include "bhq_sort.h"

// No contraction into fused multiply-adds: every kernel that locates a
// particle's mesh cell must get the bits the sort keys were made with.
#pragma clang fp contract(off)

namespace {

constexpr int kBlock = 256;
constexpr double kPi = 3.14159265358979323846;

inline unsigned nblocks(int64_t n) { return (unsigned)((n + kBlock - 1) / kBlock); }

struct Tsc {
    int i[3];        // nearest mesh index per axis (already mod n)
    double w[3][3];  // weights for offsets -1, 0, +1 per axis
};

// Offset of coordinate x from its nearest mesh point, in mesh spacings.
__device__ __forceinline__ double tsc_d(double x, double ih, double &i0)
{
    const double u = x * ih;
    i0 = floor(u + 0.5);
    return u - i0;
}

// TSC weight of the mesh point at offset o (-1, 0, +1) for offset d.
__device__ __forceinline__ double tsc_w(double d, int o)
{
    return o < 0 ? 0.5 * (0.5 - d) * (0.5 - d)
                 : (o == 0 ? 0.75 - d * d : 0.5 * (0.5 + d) * (0.5 + d));
}

__device__ __forceinline__ Tsc tsc(const double *x, double ih, int n)
{
    Tsc t;
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        double i0;
        const double d = tsc_d(x[a], ih, i0);
        // i0 mod n; positions inside the box need no division
        int64_t k = (int64_t)i0;
        if (k < 0 || k >= n) {
            k %= n;
            if (k < 0) k += n;
        }
        t.i[a] = (int)k;
        t.w[0][a] = tsc_w(d, -1);
        t.w[1][a] = tsc_w(d, 0);
        t.w[2][a] = tsc_w(d, 1);
    }
    return t;
}

__device__ __forceinline__ int wrap(int i, int n) { return i < 0 ? i + n : (i >= n ? i - n : i); }

// i mod n in [0, n) for any i (meshes smaller than a tile wrap several times)
__device__ __forceinline__ int pmod(int i, int n)
{
    const int r = i % n;
    return r < 0 ? r + n : r;
}

// Tiles of the mesh (cells of the interpolation): kTX x kTY x kTZ per block
// of kBlock threads, z fastest; with their neighbours, kHX x kHY x kHZ.
// Interpolation on 256^3 / 128^3 points by tile: 2 x 8 x 16 1.10 / 0.134 ms,
// 2 x 8 x 32 1.25 / 0.131, 4 x 4 x 32 1.04 / 0.127, 4 x 8 x 16 1.03 / 0.130
// (under the tracer).
constexpr int kXcds = 8;
constexpr int kTX = 4, kTY = 8, kTZ = 16;
constexpr int kHX = kTX + 2, kHY = kTY + 2, kHZ = kTZ + 2;
constexpr int kHalo = kHX * kHY * kHZ;
constexpr int kRows = kTX * kTY;
static_assert(kRows <= 64, "a wave scans the rows");

inline unsigned ntiles(int n)
{
    const int t = ((n + kTX - 1) / kTX) * ((n + kTY - 1) / kTY) * ((n + kTZ - 1) / kTZ);
    return (unsigned)((t + kXcds - 1) / kXcds * kXcds);
}

// Origin of the block's tile (x0 >= n: none).  Blocks go to the XCDs round
// robin; each takes a run of consecutive tiles, whose neighbourhoods overlap
// in its L2.
__device__ __forceinline__ void tile_origin(int n, int &x0, int &y0, int &z0)
{
    const int nz = (n + kTZ - 1) / kTZ, ny = (n + kTY - 1) / kTY;
    const int per = (int)(gridDim.x / kXcds);
    int b = (int)(blockIdx.x % kXcds) * per + (int)(blockIdx.x / kXcds);
    z0 = (b % nz) * kTZ;
    b /= nz;
    y0 = (b % ny) * kTY;
    x0 = (b / ny) * kTX;
}

// Mesh index of neighbourhood entry h of the tile at (x0, y0, z0).
__device__ __forceinline__ int64_t halo_point(int h, int n, int x0, int y0, int z0)
{
    const int hz = h % kHZ, hy = (h / kHZ) % kHY, hx = h / (kHZ * kHY);
    const int cx = pmod(x0 - 1 + hx, n), cy = pmod(y0 - 1 + hy, n), cz = pmod(z0 - 1 + hz, n);
    return ((int64_t)cx * n + cy) * n + cz;
}

// Cell of the particle's nearest mesh point.
struct CellKeys {
    const double *x;
    double ih;
    int n;

    __device__ __forceinline__ uint32_t operator()(int64_t p) const
    {
        const Tsc t = tsc(x + 3 * p, ih, n);
        return (uint32_t)(((int64_t)t.i[0] * n + t.i[1]) * n + t.i[2]);
    }
};

// The cells, and the identity order.
__global__ __launch_bounds__(kBlock) void k_cell_keys(int64_t np, const CellKeys keys,
                                                      uint32_t *key, int32_t *idx)
{
    const int64_t p = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (p >= np) return;
    key[p] = keys(p);
    idx[p] = (int32_t)p;
}

// Sorted particle records (x, y, z, m) and first[c] = first sorted particle of
// cell c or later (first[n3] = np), written by the particle at whose key the
// range of cells ends.  Long ranges of empty cells are written by the whole
// wave.  Also clears the count of k_rho's crowded blocks.
__global__ __launch_bounds__(kBlock) void k_sorted(int64_t np, int64_t n3, const uint32_t *key,
                                                   const int32_t *idx, const double *x,
                                                   const double *m, double4 *xs,
                                                   int32_t *first, int32_t *crowded)
{
    const int64_t k = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (k == 0) *crowded = 0;
    int64_t lo = 0, hi = -1;  // cells lo .. hi begin at k
    if (k <= np) {
        lo = k > 0 ? (int64_t)key[k - 1] + 1 : 0;
        hi = k < np ? (int64_t)key[k] : n3;
    }
    if (k < np) {
        const int64_t p = idx[k];
        xs[k] = make_double4(x[3 * p], x[3 * p + 1], x[3 * p + 2], m[p]);
    }
    constexpr int64_t kOwn = 8;
    const bool small = hi - lo < kOwn;
    if (small)
        for (int64_t c = lo; c <= hi; ++c) first[c] = (int32_t)k;
    uint64_t left = __ballot(!small);
    while (left) {
        const int l = __builtin_ctzll(left);
        left &= left - 1;
        const int64_t a = __shfl(lo, l), b = __shfl(hi, l), v = __shfl(k, l);
        for (int64_t c = a + (threadIdx.x & 63); c <= b; c += 64) first[c] = (int32_t)v;
    }
}

// rho at a mesh point: the particles whose nearest point is one of the 27
// around it, each with its TSC weight, in a fixed order: plane by plane in
// x, row by row in y, and the three z-cells of a row (whose particles are
// contiguous) in the sorted order.
// A block takes kRY x kRZ columns of mesh points, a thread each, and `len` of
// their points: it goes over the planes of cells, keeping the sums of the
// three points that a plane's particles reach, so that a particle is visited
// once for all three.  A plane's particles (of the tile's cells and their
// neighbours, 324 cells) go to LDS with their weights, computed once per
// plane, in parts of kPlaneCap.  A thread per mesh point that visited a
// particle and formed its weights for each of the 27 took 1.18 ms on 2^24
// particles and 256^3 points and 0.156 on 2,000,003 and 128^3 (VALU); this
// takes 0.60 and 0.079.
constexpr int kRY = 16, kRZ = 16;
constexpr int kPY = kRY + 2, kPZ = kRZ + 2;
constexpr int kPlane = kPY * kPZ;
constexpr int kPlaneCap = 448;
static_assert(kRY * kRZ == kBlock, "a column per thread");

// A thread goes over the particles of its cells one by one, so a block is as
// long as its fullest cells: a block with a cell of more than kCrowded
// particles among those it looks at leaves its points to k_rho_crowded
// (crowded[0] counts such blocks, their numbers follow).  Whole evaluations
// (ms) with every block here, with 16, 24 and 32, and with a thread per mesh
// point over its 27 cells: Plummer spheres of scale 0.05 in the box, 2,000,003
// particles on 128^3 56 / 2.1 / 2.2 / 2.3 / 15; 0.1, 4,000,000 on 256^3 8.7 / 3.1 /
// 3.3 / 3.7 / 5.1; uniform particles, 8 per point on 128^3 3.5 / 5.6 / 3.5 / 3.5 / 5.6, 16
// on 64^3 1.33 / 1.12 / 1.12 / 1.41 / 1.42, 64 10.0 / 4.1 / 4.1 / 4.1 / 7.3.
constexpr int kCrowded = 24;

inline unsigned rho_blocks(int n, int len)
{
    return (unsigned)(((n + kRY - 1) / kRY) * ((n + kRZ - 1) / kRZ) * ((n + len - 1) / len));
}

// Points per column and block: eight, or fewer where the blocks would not fill
// the chip (each costs two planes more than it has points).
inline int rho_len(int n)
{
    int len = 8;
    while (len > 2 && rho_blocks(n, len) < 1024) len /= 2;
    return len;
}

// First mesh point of block b.
__device__ __forceinline__ void rho_origin(int b, int n, int len, int &x0, int &y0, int &z0)
{
    const int nz = (n + kRZ - 1) / kRZ, ny = (n + kRY - 1) / kRY;
    z0 = (b % nz) * kRZ;
    b /= nz;
    y0 = (b % ny) * kRY;
    x0 = (b / ny) * len;
}

__global__ __launch_bounds__(kBlock) void k_rho(int n, double ih, int len, const double4 *xs,
                                                const int32_t *first, double *rho,
                                                int32_t *crowded)
{
    typedef hipcub::BlockScan<int, kBlock> Scan;
    __shared__ double mwx[3][kPlaneCap], wy[3][kPlaneCap], wz[3][kPlaneCap];
    __shared__ int32_t sfirst[kPlane + 1], sstart[kPlane];
    __shared__ typename Scan::TempStorage scan_tmp;
    int x0, y0, z0;
    rho_origin((int)blockIdx.x, n, len, x0, y0, z0);
    const int t = threadIdx.x, tz = t % kRZ, ty = t / kRZ;
    const int xe = x0 + len < n ? x0 + len : n;
    constexpr int kPer = (kPlane + kBlock - 1) / kBlock;
    // mesh row and column of the cells that this thread counts (row < 0: none;
    // on a mesh smaller than the tile those around its points are enough)
    int row[kPer], col[kPer];
#pragma unroll
    for (int u = 0; u < kPer; ++u) {
        const int h = kPer * t + u, hy = h / kPZ, hz = h % kPZ;
        const bool use = h < kPlane && hy < n + 2 && hz < n + 2;
        row[u] = use ? pmod(y0 - 1 + hy, n) : -1;
        col[u] = use ? pmod(z0 - 1 + hz, n) : 0;
    }
    double s0 = 0.0, s1 = 0.0, s2 = 0.0;  // points px - 1, px, px + 1
    for (int px = x0 - 1; px <= xe; ++px) {
        const int64_t plane = (int64_t)pmod(px, n) * n;
        int cnt[kPer], part = 0;
        bool full = false;
#pragma unroll
        for (int u = 0; u < kPer; ++u) {
            const int h = kPer * t + u;
            cnt[u] = 0;
            if (row[u] >= 0) {
                const int64_t c = (plane + row[u]) * n + col[u];
                const int32_t f = first[c];
                cnt[u] = first[c + 1] - f;
                sstart[h] = f;
            }
            part += cnt[u];
            full |= cnt[u] > kCrowded;
        }
        int at = 0, total = 0;
        Scan(scan_tmp).ExclusiveSum(part, at, total);
#pragma unroll
        for (int u = 0; u < kPer; ++u) {
            const int h = kPer * t + u;
            if (h < kPlane) sfirst[h] = at;
            at += cnt[u];
        }
        if (t == 0) sfirst[kPlane] = total;
        if (__syncthreads_or(full)) {
            if (t == 0) crowded[1 + atomicAdd(crowded, 1)] = (int32_t)blockIdx.x;
            return;
        }
        for (int c0 = 0; c0 < total; c0 += kPlaneCap) {
            const int c1 = total - c0 < kPlaneCap ? total : c0 + kPlaneCap;
            if (c0 > 0) __syncthreads();
            for (int j = c0 + t; j < c1; j += kBlock) {
                // the last cell whose first entry is j or before
                int lo = 0, hi = kPlane;
                while (hi - lo > 1) {
                    const int mid = (lo + hi) >> 1;
                    if (sfirst[mid] <= j)
                        lo = mid;
                    else
                        hi = mid;
                }
                const double4 r = xs[sstart[lo] + (j - sfirst[lo])];
                double i0;
                const double dx = tsc_d(r.x, ih, i0), dy = tsc_d(r.y, ih, i0),
                             dz = tsc_d(r.z, ih, i0);
#pragma unroll
                for (int o = -1; o <= 1; ++o) {
                    mwx[o + 1][j - c0] = r.w * tsc_w(dx, o);
                    wy[o + 1][j - c0] = tsc_w(dy, o);
                    wz[o + 1][j - c0] = tsc_w(dz, o);
                }
            }
            __syncthreads();
            // rows of cells below, at and above the thread's points in y are at
            // offsets +1, 0, -1 from their particles; in z the same
#pragma unroll
            for (int q = 0; q < 3; ++q) {
                const int h0 = (ty + q) * kPZ + tz;
                const int f0 = sfirst[h0], f1 = sfirst[h0 + 1], f2 = sfirst[h0 + 2],
                          f3 = sfirst[h0 + 3];
                const int ka = f0 > c0 ? f0 : c0, kb = f3 < c1 ? f3 : c1;
                for (int k = ka; k < kb; ++k) {
                    const int o = 2 - (k >= f1 ? 1 : 0) - (k >= f2 ? 1 : 0);
                    const int j = k - c0;
                    const double w = wy[2 - q][j] * wz[o][j];
                    s0 = fma(mwx[0][j], w, s0);
                    s1 = fma(mwx[1][j], w, s1);
                    s2 = fma(mwx[2][j], w, s2);
                }
            }
        }
        const int qy = y0 + ty, qz = z0 + tz;
        if (px > x0 && qy < n && qz < n) rho[((int64_t)(px - 1) * n + qy) * n + qz] = s0;
        s0 = s1;
        s1 = s2;
        s2 = 0.0;
        __syncthreads();
    }
}

// TSC weight for offset o (-1, 0, +1) with o known only at run time; the
// same operations as tsc_w (negating d is exact).
__device__ __forceinline__ double tsc_w_var(double d, int o)
{
    const double s = o < 0 ? -d : d;
    return o == 0 ? 0.75 - d * d : 0.5 * (0.5 + s) * (0.5 + s);
}

__device__ __forceinline__ double tsc_offset(double x, double ih)
{
    double i0;
    return tsc_d(x, ih, i0);
}

// rho at the points of the crowded blocks, a wave per point: lane c < 27
// finds the range of cell c around the point, the lanes go side by side over
// the particles of all of them, and the lanes' sums are added in a fixed
// order.  However the particles are concentrated, the work is spread over the
// points that they reach.
constexpr int kCrowdedBlocks = 1024;

__global__ __launch_bounds__(kBlock) void k_rho_crowded(int n, double ih, int len,
                                                        const double4 *xs, const int32_t *first,
                                                        const int32_t *crowded, double *rho)
{
    const int lane = threadIdx.x & 63;
    const int per = kBlock * len;  // points of a block of k_rho
    const int64_t points = (int64_t)crowded[0] * per;
    constexpr int kWaves = kCrowdedBlocks * (kBlock / 64);
    for (int64_t i = blockIdx.x * (kBlock / 64) + threadIdx.x / 64; i < points; i += kWaves) {
        int x0, y0, z0;
        rho_origin(crowded[1 + i / per], n, len, x0, y0, z0);
        const int r = (int)(i % per);
        const int px = x0 + r / kBlock, py = y0 + r % kBlock / kRZ, pz = z0 + r % kRZ;
        if (px >= n || py >= n || pz >= n) continue;
        int32_t lo = 0, incl = 0;
        if (lane < 27) {
            const int64_t c = ((int64_t)wrap(px + lane / 9 - 1, n) * n +
                               wrap(py + lane / 3 % 3 - 1, n)) * n + wrap(pz + lane % 3 - 1, n);
            lo = first[c];
            incl = first[c + 1] - lo;
        }
        const int own = incl;
        for (int h = 1; h < 32; h *= 2) {
            const int v = __shfl_up(incl, h);
            if (lane >= h) incl += v;
        }
        lo -= incl - own;  // sorted index of cell c's particle j: lo + j
        const int total = __shfl(incl, 26);
        double s = 0.0;
        for (int j = lane; j - lane < total; j += 64) {
            int c = 0;  // cells that end at or before j
            for (int h = 16; h > 0; h /= 2)
                if (__shfl(incl, c + h - 1) <= j) c += h;
            c = c < 26 ? c : 26;
            const int64_t k = (int64_t)__shfl(lo, c) + j;
            if (j < total) {
                const double4 q = xs[k];
                // a cell below the point is at offset +1 from its particles
                const double wx = tsc_w_var(tsc_offset(q.x, ih), 1 - c / 9),
                             wy = tsc_w_var(tsc_offset(q.y, ih), 1 - c / 3 % 3),
                             wz = tsc_w_var(tsc_offset(q.z, ih), 1 - c % 3);
                s = fma(q.w * wx, wy * wz, s);
            }
        }
        for (int h = 32; h > 0; h /= 2) s += __shfl_xor(s, h);
        if (lane == 0) rho[((int64_t)px * n + py) * n + pz] = s;
    }
}

__device__ __forceinline__ double sinc_half(double kh)
{
    // sin(kh/2) / (kh/2), 1 at k = 0
    const double t = 0.5 * kh;
    return t == 0.0 ? 1.0 : sin(t) / t;
}

// rk: n x n x (n/2+1) complex; writes the three gradient arrays and phi, nc
// apart.
__global__ __launch_bounds__(kBlock) void k_green(const hipfftDoubleComplex *rk, int n,
                                                  double L, double rs, double scale,
                                                  hipfftDoubleComplex *fk)
{
    const int nz = n / 2 + 1;
    const int64_t nc = (int64_t)n * n * nz;
    const int64_t e = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (e >= (int64_t)n * n * nz) return;
    const int iz = (int)(e % nz);
    const int iy = (int)((e / nz) % n);
    const int ix = (int)(e / ((int64_t)nz * n));
    const double dk = 2.0 * kPi / L, h = L / n;
    // signed frequencies: index i < n/2 is i, the rest i - n (n/2 is -n/2)
    const double kxs = dk * (ix < n / 2 ? ix : ix - n);
    const double kys = dk * (iy < n / 2 ? iy : iy - n);
    const double kz = dk * iz;
    const double k2 = kxs * kxs + kys * kys + kz * kz;
    double g = 0.0;
    if (k2 > 0.0) {
        const double w = sinc_half(kxs * h) * sinc_half(kys * h) * sinc_half(kz * h);
        const double w3 = w * w * w;
        g = -4.0 * kPi * exp(-k2 * rs * rs) / k2 / (w3 * w3) * scale;
    }
    const hipfftDoubleComplex r = rk[e];
    const double pr = g * r.x, pi = g * r.y;
    fk[3 * nc + e] = make_hipDoubleComplex(pr, pi);
    // -i k phi = (k phi_i, -k phi_r)
    const double gx = ix == n / 2 ? 0.0 : kxs;
    const double gy = iy == n / 2 ? 0.0 : kys;
    const double gz = iz == n / 2 ? 0.0 : kz;
    fk[e] = make_hipDoubleComplex(gx * pi, -gx * pr);
    fk[nc + e] = make_hipDoubleComplex(gy * pi, -gy * pr);
    fk[2 * nc + e] = make_hipDoubleComplex(gz * pi, -gz * pr);
}

// One term of the 27-point interpolation, in the order of the points.
__device__ __forceinline__ void interp_add(const Tsc &w, int a0, int b, int c, const double4 &v,
                                           double *s4)
{
    const double wt = w.w[a0][0] * w.w[b][1] * w.w[c][2];
    s4[0] = fma(wt, v.x, s4[0]);
    s4[1] = fma(wt, v.y, s4[1]);
    s4[2] = fma(wt, v.z, s4[2]);
    s4[3] = fma(wt, v.w, s4[3]);
}

// The particles of the block's tile of cells (nearest mesh point in the
// tile; a row of the tile along z is a contiguous range of the sorted
// order): 27-point TSC interpolation of the four meshes (a_x, a_y, a_z, phi,
// n3 apart), whose values around the tile are in LDS as one record per point;
// each result goes to the particle's input index.
// A block is one chain of loads (rows, particles, fields): each wave finds
// the rows' ranges itself, by shuffles, and the particles are loaded before
// the fields, so that only the fields are waited for together.  With ranges
// from LDS atomics, a serial sum of them and a separate pass that interleaved
// the meshes this took 1.17 ms on 2^24 particles and 256^3 points, now 0.92
// (0.157 and 0.130 on 2,000,003 unsorted particles and 128^3).  What is left
// are the neighbourhoods (2.1 mesh points read per point of the tile) and
// their reads from LDS.
__global__ __launch_bounds__(kBlock) void k_interp(int n, const double4 *xs, const int32_t *idx,
                                                   const int32_t *first, double ih,
                                                   const double *mesh, int64_t n3, double *a,
                                                   double *pot, int accumulate)
{
    __shared__ double4 sm[kHalo];
    int x0, y0, z0;
    tile_origin(n, x0, y0, z0);
    if (x0 >= n) return;
    const int t = threadIdx.x, lane = t & 63;
    // lane r: range and inclusive count of row r's particles
    int32_t lo = 0, incl = 0;
    {
        const int cx = x0 + lane / kTY, cy = y0 + lane % kTY;
        if (lane < kRows && cx < n && cy < n) {
            const int64_t c = ((int64_t)cx * n + cy) * n + z0;
            lo = first[c];
            incl = first[c + (n - z0 < kTZ ? n - z0 : kTZ)] - lo;
        }
        for (int h = 1; h < kRows; h *= 2) {
            const int v = __shfl_up(incl, h);
            if (lane >= h) incl += v;
        }
    }
    const int total = __shfl(incl, kRows - 1);
    // sorted index of the tile's particle j
    auto sorted_index = [&](int j) -> int64_t {
        int r = 0;  // rows that end at or before j
        for (int h = kRows / 2; h > 0; h /= 2)
            if (__shfl(incl, r + h - 1) <= j) r += h;
        const int before = __shfl(incl, r > 0 ? r - 1 : 0);
        return (int64_t)__shfl(lo, r) + (j - (r > 0 ? before : 0));
    };
    double4 rec = make_double4(0.0, 0.0, 0.0, 0.0);
    int64_t p = 0;
    {
        const int64_t k = sorted_index(t < total ? t : 0);
        if (t < total) {
            rec = xs[k];
            p = idx[k];
        }
    }
    for (int h = t; h < kHalo; h += kBlock) {
        const int64_t q = halo_point(h, n, x0, y0, z0);
        sm[h] = make_double4(mesh[q], mesh[n3 + q], mesh[2 * n3 + q], mesh[3 * n3 + q]);
    }
    __syncthreads();
    for (int j = t; j - lane < total; j += kBlock) {
        if (j >= kBlock) {
            const int64_t k = sorted_index(j < total ? j : 0);
            if (j < total) {
                rec = xs[k];
                p = idx[k];
            }
        }
        if (j >= total) break;
        const double xp[3] = {rec.x, rec.y, rec.z};
        const Tsc w = tsc(xp, ih, n);
        // the particle's cell is in the tile (its sort key was computed by
        // the same function): its neighbourhood entries are (w.i - origin) +
        // (0 .. 2) per axis; a cell outside the tile would read the mesh
        const int hx0 = w.i[0] - x0, hy0 = w.i[1] - y0, hz0 = w.i[2] - z0;
        const bool in = hx0 >= 0 && hx0 < kTX && hy0 >= 0 && hy0 < kTY && hz0 >= 0 &&
                        hz0 < kTZ;
        double s4[4] = {0.0, 0.0, 0.0, 0.0};
        if (in) {
#pragma unroll
            for (int a0 = 0; a0 < 3; ++a0)
#pragma unroll
                for (int b = 0; b < 3; ++b)
#pragma unroll
                    for (int c = 0; c < 3; ++c)
                        interp_add(w, a0, b, c,
                                   sm[((hx0 + a0) * kHY + (hy0 + b)) * kHZ + (hz0 + c)], s4);
        } else {
            for (int a0 = 0; a0 < 3; ++a0)
                for (int b = 0; b < 3; ++b)
                    for (int c = 0; c < 3; ++c) {
                        const int64_t q = ((int64_t)wrap(w.i[0] + a0 - 1, n) * n +
                                           wrap(w.i[1] + b - 1, n)) * n +
                                          wrap(w.i[2] + c - 1, n);
                        const double wt = tsc_w_var(tsc_offset(xp[0], ih), a0 - 1) *
                                          tsc_w_var(tsc_offset(xp[1], ih), b - 1) *
                                          tsc_w_var(tsc_offset(xp[2], ih), c - 1);
                        for (int f = 0; f < 4; ++f) s4[f] = fma(wt, mesh[f * n3 + q], s4[f]);
                    }
        }
        if (accumulate) {
            a[3 * p] += s4[0];
            a[3 * p + 1] += s4[1];
            a[3 * p + 2] += s4[2];
            if (pot) pot[p] += s4[3];
        } else {
            a[3 * p] = s4[0];
            a[3 * p + 1] = s4[1];
            a[3 * p + 2] = s4[2];
            if (pot) pot[p] = s4[3];
        }
    }
}

}  // namespace

// Largest mesh whose inverse transforms are batched.
constexpr int kBatchMesh = 224;

struct bhq_pm {
    int device = 0;
    int n = 0;
    double box = 0.0, rs = 0.0;
    std::string err;
    bhq::DevArray rho, rk, fk, mesh;  // fk, mesh: four fields each
    // per-particle sorting (grown to the largest n seen)
    bhq::DevArray key, key2, idx, idx2, xs, sort_tmp, first;
    bhq::DevArray crowded;  // k_rho's crowded blocks: count, numbers
    hipfftHandle fwd = 0, inv = 0;
    int batch = 1;  // fields per inverse transform
    bool have_fwd = false, have_inv = false;
    hipEvent_t ev0 = nullptr, ev1 = nullptr;
    bool launched = false;

    int fail(int code, const char *fmt, ...)
    {
        char buf[512];
        va_list ap;
        va_start(ap, fmt);
        vsnprintf(buf, sizeof(buf), fmt, ap);
        va_end(ap);
        err = buf;
        return code;
    }
};

namespace {

thread_local std::string g_pm_create_error;

void pm_free(bhq_pm *p)
{
    if (p->have_fwd) (void)hipfftDestroy(p->fwd);
    if (p->have_inv) (void)hipfftDestroy(p->inv);
    for (bhq::DevArray *a : {&p->rho, &p->rk, &p->fk, &p->mesh, &p->key, &p->key2, &p->idx,
                             &p->idx2, &p->xs, &p->sort_tmp, &p->first, &p->crowded})
        a->release();
    if (p->ev0) (void)hipEventDestroy(p->ev0);
    if (p->ev1) (void)hipEventDestroy(p->ev1);
    delete p;
}

int check_range(bhq_pm *pm, const void *ptr, size_t bytes, const char *name)
{
    hipDeviceptr_t base = nullptr;
    size_t size = 0;
    if (hipMemGetAddressRange(&base, &size, const_cast<void *>(ptr)) != hipSuccess || !base) {
        (void)hipGetLastError();
        return pm->fail(BHQ_E_ARG, "%s is not device memory", name);
    }
    const char *b = static_cast<const char *>(base);
    const char *q = static_cast<const char *>(ptr);
    if (q < b || (size_t)(q - b) + bytes > size)
        return pm->fail(BHQ_E_RANGE, "%s: %zu bytes do not fit its allocation", name, bytes);
    return BHQ_OK;
}

}  // namespace

extern "C" {

int bhq_pm_create(bhq_pm **out, int device, int nmesh, double box, double rs)
{
    if (!out) return BHQ_E_ARG;
    *out = nullptr;
    if (nmesh < 4 || nmesh > 1024 || (nmesh & 1) || !(box > 0.0) || !std::isfinite(box) ||
        !(rs > 0.0) || !std::isfinite(rs)) {
        g_pm_create_error = "bhq_pm_create: need an even mesh size in [4, 1024], box > 0, rs > 0";
        return BHQ_E_ARG;
    }
    int count = 0;
    if (hipGetDeviceCount(&count) != hipSuccess || device < 0 || device >= count) {
        g_pm_create_error = "bhq_pm_create: no such device";
        return BHQ_E_NODEV;
    }
    if (hipSetDevice(device) != hipSuccess) {
        g_pm_create_error = "bhq_pm_create: hipSetDevice failed";
        return BHQ_E_HIP;
    }
    bhq_pm *p = new (std::nothrow) bhq_pm();
    if (!p) {
        g_pm_create_error = "bhq_pm_create: out of host memory";
        return BHQ_E_NOMEM;
    }
    p->device = device;
    p->n = nmesh;
    p->box = box;
    p->rs = rs;
    const size_t n3 = (size_t)nmesh * nmesh * nmesh;
    const size_t nc = (size_t)nmesh * nmesh * (nmesh / 2 + 1);
    hipError_t e = hipSuccess;
    e = p->rho.reserve(n3 * sizeof(double));
    if (e == hipSuccess) e = p->rk.reserve(nc * sizeof(hipfftDoubleComplex));
    if (e == hipSuccess) e = p->fk.reserve(4 * nc * sizeof(hipfftDoubleComplex));
    if (e == hipSuccess) e = p->mesh.reserve(4 * n3 * sizeof(double));
    if (e == hipSuccess) e = p->first.reserve((n3 + 1) * sizeof(int32_t));
    if (e == hipSuccess)
        e = p->crowded.reserve((rho_blocks(nmesh, rho_len(nmesh)) + 1) * sizeof(int32_t));
    if (e == hipSuccess) e = hipEventCreate(&p->ev0);
    if (e == hipSuccess) e = hipEventCreate(&p->ev1);
    if (e != hipSuccess) {
        g_pm_create_error = std::string("bhq_pm_create: ") + hipGetErrorString(e);
        const int code = (e == hipErrorOutOfMemory) ? BHQ_E_NOMEM : BHQ_E_HIP;
        pm_free(p);
        return code;
    }
    if (hipfftPlan3d(&p->fwd, nmesh, nmesh, nmesh, HIPFFT_D2Z) != HIPFFT_SUCCESS) {
        g_pm_create_error = "bhq_pm_create: hipFFT forward plan failed";
        pm_free(p);
        return BHQ_E_HIP;
    }
    p->have_fwd = true;
    // The four inverse transforms go in one batch as far as that is faster:
    // whole evaluations with few particles, one after another / together (us),
    // 60^3 141 / 108, 128^3 308 / 257, 130^3 403 / 333, 160^3 506 / 459, 192^3 834 / 782,
    // 224^3 1183 / 1141, 256^3 1807 / 1808.  From there on they are equal within 2 %, and
    // one after another they need a quarter of the work memory.
    p->batch = nmesh <= kBatchMesh ? 4 : 1;
    int dims[3] = {nmesh, nmesh, nmesh};
    if (hipfftPlanMany(&p->inv, 3, dims, nullptr, 1, 0, nullptr, 1, 0, HIPFFT_Z2D, p->batch) !=
        HIPFFT_SUCCESS) {
        g_pm_create_error = "bhq_pm_create: hipFFT inverse plan failed";
        pm_free(p);
        return BHQ_E_HIP;
    }
    p->have_inv = true;
    g_pm_create_error.clear();
    *out = p;
    return BHQ_OK;
}

int bhq_pm_destroy(bhq_pm *pm)
{
    if (!pm) return BHQ_OK;
    (void)hipSetDevice(pm->device);
    if (pm->launched) (void)hipEventSynchronize(pm->ev1);
    pm_free(pm);
    return BHQ_OK;
}

int bhq_pm_compute(bhq_pm *pm, int64_t np, const double *x, const double *m, double *a,
                   double *pot, int accumulate, void *stream)
{
    if (!pm) return BHQ_E_ARG;
    if (np < 1 || np > 0x7fffffffLL || !x || !m || !a || (accumulate != 0 && accumulate != 1))
        return pm->fail(BHQ_E_ARG, "pm_compute: bad argument");
    if (hipSetDevice(pm->device) != hipSuccess) return pm->fail(BHQ_E_HIP, "hipSetDevice");
    int rc = check_range(pm, x, (size_t)np * 3 * sizeof(double), "x");
    if (rc == BHQ_OK) rc = check_range(pm, m, (size_t)np * sizeof(double), "m");
    if (rc == BHQ_OK) rc = check_range(pm, a, (size_t)np * 3 * sizeof(double), "a");
    if (rc == BHQ_OK && pot) rc = check_range(pm, pot, (size_t)np * sizeof(double), "pot");
    if (rc != BHQ_OK) return rc;
    hipStream_t s = static_cast<hipStream_t>(stream);
    const int n = pm->n;
    const double h = pm->box / n, ih = 1.0 / h;
    const size_t n3 = (size_t)n * n * n;
    const int64_t nc = (int64_t)n * n * (n / 2 + 1);
    // density = mass / h^3; the inverse transforms are unnormalised (1/n^3)
    const double scale = 1.0 / (h * h * h) / (double)n3;
    auto hipok = [&](hipError_t e, const char *w) -> bool {
        if (e == hipSuccess) return true;
        pm->fail(BHQ_E_HIP, "pm_compute: %s: %s", w, hipGetErrorString(e));
        return false;
    };
    auto fftok = [&](hipfftResult r, const char *w) -> bool {
        if (r == HIPFFT_SUCCESS) return true;
        pm->fail(BHQ_E_HIP, "pm_compute: %s failed (hipFFT %d)", w, (int)r);
        return false;
    };
    if (!hipok(hipEventRecord(pm->ev0, s), "event")) return BHQ_E_HIP;
    // particles sorted by their nearest mesh point, cell ranges, density
    for (bhq::DevArray *b : {&pm->key, &pm->key2})
        if (!hipok(b->reserve((size_t)np * 4), "allocation")) return BHQ_E_NOMEM;
    for (bhq::DevArray *b : {&pm->idx, &pm->idx2})
        if (!hipok(b->reserve((size_t)np * 4), "allocation")) return BHQ_E_NOMEM;
    if (!hipok(pm->xs.reserve((size_t)np * sizeof(double4)), "allocation")) return BHQ_E_NOMEM;
    int bits = 1;
    while (((uint64_t)1 << bits) < (uint64_t)n3) ++bits;
    const CellKeys keys{x, ih, n};
    uint32_t *k0 = pm->key.as<uint32_t>(), *k1 = pm->key2.as<uint32_t>();
    int32_t *i0 = pm->idx.as<int32_t>(), *i1 = pm->idx2.as<int32_t>();
    if (np <= bhq::kRankSortMost && bits < 32) {
        if (!hipok(bhq::rank_sort(keys, np, 0, bits, k0, i0, k1, i1, s), "sort"))
            return BHQ_E_HIP;
    } else {
        size_t tmp = 0;
        if (!hipok(hipcub::DeviceRadixSort::SortPairs(nullptr, tmp, k0, k1, i0, i1, (int)np, 0,
                                                      bits, s),
                   "sort size"))
            return BHQ_E_HIP;
        if (!hipok(pm->sort_tmp.reserve(tmp), "allocation")) return BHQ_E_NOMEM;
        hipLaunchKernelGGL(k_cell_keys, dim3(nblocks(np)), dim3(kBlock), 0, s, np, keys, k0, i0);
        if (!hipok(hipGetLastError(), "cell keys")) return BHQ_E_HIP;
        if (!hipok(hipcub::DeviceRadixSort::SortPairs(pm->sort_tmp.p, tmp, k0, k1, i0, i1,
                                                      (int)np, 0, bits, s),
                   "sort"))
            return BHQ_E_HIP;
    }
    hipLaunchKernelGGL(k_sorted, dim3(nblocks(np + 1)), dim3(kBlock), 0, s, np, (int64_t)n3,
                       pm->key2.as<uint32_t>(), pm->idx2.as<int32_t>(), x, m,
                       pm->xs.as<double4>(), pm->first.as<int32_t>(),
                       pm->crowded.as<int32_t>());
    if (!hipok(hipGetLastError(), "sorted records")) return BHQ_E_HIP;
    const int len = rho_len(n);
    hipLaunchKernelGGL(k_rho, dim3(rho_blocks(n, len)), dim3(kBlock), 0, s, n, ih, len,
                       pm->xs.as<double4>(), pm->first.as<int32_t>(), pm->rho.as<double>(),
                       pm->crowded.as<int32_t>());
    if (!hipok(hipGetLastError(), "assignment")) return BHQ_E_HIP;
    hipLaunchKernelGGL(k_rho_crowded, dim3(kCrowdedBlocks), dim3(kBlock), 0, s, n, ih, len,
                       pm->xs.as<double4>(), pm->first.as<int32_t>(),
                       pm->crowded.as<int32_t>(), pm->rho.as<double>());
    if (!hipok(hipGetLastError(), "assignment")) return BHQ_E_HIP;
    if (!fftok(hipfftSetStream(pm->fwd, s), "set stream") ||
        !fftok(hipfftSetStream(pm->inv, s), "set stream"))
        return BHQ_E_HIP;
    if (!fftok(hipfftExecD2Z(pm->fwd, pm->rho.as<hipfftDoubleReal>(),
                             pm->rk.as<hipfftDoubleComplex>()),
               "forward FFT"))
        return BHQ_E_HIP;
    hipLaunchKernelGGL(k_green, dim3(nblocks(nc)), dim3(kBlock), 0, s,
                       pm->rk.as<hipfftDoubleComplex>(), n, pm->box, pm->rs, scale,
                       pm->fk.as<hipfftDoubleComplex>());
    if (!hipok(hipGetLastError(), "green function")) return BHQ_E_HIP;
    for (int f = 0; f < 4; f += pm->batch)
        if (!fftok(hipfftExecZ2D(pm->inv, pm->fk.as<hipfftDoubleComplex>() + f * nc,
                                 pm->mesh.as<hipfftDoubleReal>() + f * (int64_t)n3),
                   "inverse FFT"))
            return BHQ_E_HIP;
    hipLaunchKernelGGL(k_interp, dim3(ntiles(n)), dim3(kBlock), 0, s, n, pm->xs.as<double4>(),
                       pm->idx2.as<int32_t>(), pm->first.as<int32_t>(), ih,
                       pm->mesh.as<double>(), (int64_t)n3, a, pot, accumulate);
    if (!hipok(hipGetLastError(), "interpolation")) return BHQ_E_HIP;
    if (!hipok(hipEventRecord(pm->ev1, s), "event")) return BHQ_E_HIP;
    pm->launched = true;
    return BHQ_OK;
}

int bhq_pm_get_ms(bhq_pm *pm, double *ms)
{
    if (!pm || !ms) return BHQ_E_ARG;
    if (!pm->launched) return pm->fail(BHQ_E_STATE, "pm_get_ms before compute");
    float f = 0.0f;
    if (hipEventSynchronize(pm->ev1) != hipSuccess ||
        hipEventElapsedTime(&f, pm->ev0, pm->ev1) != hipSuccess)
        return pm->fail(BHQ_E_HIP, "pm_get_ms: event query failed");
    *ms = f;
    return BHQ_OK;
}

const char *bhq_pm_last_error(const bhq_pm *pm)
{
    return pm ? pm->err.c_str() : g_pm_create_error.c_str();
}

}  // extern "C"
