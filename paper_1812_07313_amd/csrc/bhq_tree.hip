// bhq_tree.hip -- the oct-tree, its groups and the interaction lists built
// on the GPU from particles already in device memory.
//
// The construction is the host builder's (Kodama & Ishiyama, Sec. 1 for
// the tree, Sec. 3.4 for the groups and their shared lists), step by step,
// so that cells, moments, groups and lists come out identical:
//   1. root cube from the bounding box (or [0, box)^3); for a batch of
//      independent systems one root per system from that system's box;
//   2. a 63-bit key per particle by descending 21 levels (upper half along
//      an axis iff the coordinate is >= the cell centre), then a stable
//      radix sort by key (ties keep input order), system by system;
//   3. cells: a cell with more than nleaf particles above depth 21 has one
//      child per non-empty octant; all levels come from the sorted keys in
//      one pass, numbered in the order of their parents, then octants (the
//      host's breadth-first ids; a batch's system by system, the host's
//      concatenation of independently built systems); particles inside a
//      leaf return to input order;
//   4. moments: leaves from their particles, parents from their children
//      by the parallel-axis shift, deepest level first;
//   5. groups: the largest cells with at most ncrit particles (or leaves),
//      in depth-first order, which is the order of their first particle;
//   6. lists in depth-first, octant order: a block per group walks the tree
//      level by level, once to count and once to fill (a rebuild once, into
//      slots).  A cell that does not contain the group is accepted iff side^2 < theta^2 d^2 (d: its
//      centre of mass to the group cube; minimum image in a periodic box,
//      where cells farther than rcut from the group are skipped, and
//      accepted cells whose centre of mass lies at least rcut (1 + 2^-16)
//      from the bounding box of the group's particles are left out: beyond
//      the cutoff for every particle of the group).
// Every floating-point decision (key digits, acceptance) and every moment
// is computed with the host builder's operations in the same order, with
// no contraction into fused multiply-adds, so the results agree bit for
// bit.
#include <hip/hip_runtime.h>
#include <hipcub/hipcub.hpp>
#include <rocprim/rocprim.hpp>

#include <algorithm>
#include <climits>

#include "bhq.h"
#include "bhq_internal.h"
#include "bhq_sort.h"

#pragma clang fp contract(off)

namespace bhq {

namespace {

constexpr int kMaxDepth = 21;
constexpr int kFrames = kMaxDepth + 1;  // walk stack: root + one per depth
constexpr int kWalkBlock = 128;             // walk: 16 groups of 8 lanes per block
constexpr int kOct = 8;                     // lanes per group in the walk
constexpr int kXcds = 8;                    // XCDs of the chip
// walk grid: a multiple of kXcds blocks covering ng groups
inline unsigned walk_blocks(int64_t ng)
{
    const int64_t b = (ng + kWalkBlock / kOct - 1) / (kWalkBlock / kOct);
    return (unsigned)((b + kXcds - 1) / kXcds * kXcds);
}
constexpr int kBlock = 256;
constexpr int kBboxBlocks = 1024;

// A cell: geometry and centre of mass (64 B), then its particles
// [first, end) and its children [child0, cend) (child0 < 0: a leaf).
struct alignas(64) WCell {
    double cx, cy, cz, side;
    double mx, my, mz;
    double pad;
};
struct alignas(16) WLink {
    int32_t first, child0, end, cend;
};

__device__ __forceinline__ int children(const WLink &L)
{
    return L.child0 < 0 ? 0 : L.cend - L.child0;
}

inline unsigned blocks(int64_t n, int b) { return (unsigned)((n + b - 1) / b); }

// ---- 1. input check, bounding box, root cubes --------------------------------

// Minimum and maximum per axis over the block's threads: lo, hi of thread t
// in s[0..2][t], s[3..5][t]; the result in s[.][0].
template <int BS>
__device__ __forceinline__ void block_box(double (*s)[BS])
{
    __syncthreads();
    for (int h = BS / 2; h > 0; h >>= 1) {
        if ((int)threadIdx.x < h)
            for (int a = 0; a < 3; ++a) {
                const double l = s[a][threadIdx.x + h], u = s[3 + a][threadIdx.x + h];
                if (l < s[a][threadIdx.x]) s[a][threadIdx.x] = l;
                if (u > s[3 + a][threadIdx.x]) s[3 + a][threadIdx.x] = u;
            }
        __syncthreads();
    }
}

// Root cube of the box s[.][0]: centre and side, with the host builder's
// operations.
template <int BS>
__device__ __forceinline__ void root_cube(double (*s)[BS], double *root)
{
    double ext = 0.0;
    for (int a = 0; a < 3; ++a) {
        root[a] = 0.5 * (s[a][0] + s[3 + a][0]);
        const double e = s[3 + a][0] - s[a][0];
        ext = ext < e ? e : ext;
    }
    root[3] = ext > 0.0 ? ext * (1.0 + 0x1p-20) : 1.0;
}

// Per block: bad[b] bit 0 if a position or mass is not finite, bit 1 if a
// softening is not finite and positive, and with part the bounding box (one
// system).
constexpr int kFlags = 16;

__global__ __launch_bounds__(kBlock) void k_check(const double *x, const double *m,
                                                  const double *eps2, int64_t n, int *bad,
                                                  double *part)
{
    __shared__ double s[6][kBlock];
    double lo[3], hi[3];
    const int64_t start = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    const int64_t stride = (int64_t)gridDim.x * kBlock;
    const int64_t p0 = start < n ? start : 0;  // n >= 1
    for (int a = 0; a < 3; ++a) lo[a] = hi[a] = x[3 * p0 + a];
    bool input = false, soft = false;
    for (int64_t p = start; p < n; p += stride) {
        double v[3];
        for (int a = 0; a < 3; ++a) {
            v[a] = x[3 * p + a];
            lo[a] = v[a] < lo[a] ? v[a] : lo[a];
            hi[a] = v[a] > hi[a] ? v[a] : hi[a];
        }
        if (!isfinite(v[0]) || !isfinite(v[1]) || !isfinite(v[2]) || !isfinite(m[p])) input = true;
        if (eps2 && !(isfinite(eps2[p]) && eps2[p] >= kMinEps2)) soft = true;
    }
    const int f0 = __syncthreads_or(input), f1 = __syncthreads_or(soft);
    if (threadIdx.x == 0) bad[blockIdx.x] = (f0 ? 1 : 0) | (f1 ? 2 : 0);
    if (!part) return;
    for (int a = 0; a < 3; ++a) {
        s[a][threadIdx.x] = lo[a];
        s[3 + a][threadIdx.x] = hi[a];
    }
    block_box<kBlock>(s);
    if (threadIdx.x < 6) part[6 * blockIdx.x + threadIdx.x] = s[threadIdx.x][0];
}

// The build's flags from the checking blocks' (one block): flag[0], flag[1]
// as bad's bits, the others cleared.
__device__ __forceinline__ void set_flags(const int *bad, int nb, int *flag)
{
    int f = 0;
    for (int b = threadIdx.x; b < nb; b += (int)blockDim.x) f |= bad[b];
    const int f0 = __syncthreads_or(f & 1), f1 = __syncthreads_or(f & 2);
    if (threadIdx.x < kFlags)
        flag[threadIdx.x] = threadIdx.x == 0 ? (f0 ? 1 : 0) : threadIdx.x == 1 && f1 ? 1 : 0;
}

// The one system's root cube (by a block, in its LDS) from the checking
// blocks' boxes, or [0, box)^3.
__device__ __forceinline__ void one_root(const double *part, int nb, double box,
                                         double (*s)[kBlock], double *root)
{
    const int t = threadIdx.x;
    if (box > 0.0) {
        if (t < 4) root[t] = t < 3 ? 0.5 * box : box;
        __syncthreads();
        return;
    }
    const int b0 = t < nb ? t : 0;
    for (int a = 0; a < 6; ++a) s[a][t] = part[6 * b0 + a];
    for (int b = t + kBlock; b < nb; b += kBlock)
        for (int a = 0; a < 3; ++a) {
            const double l = part[6 * b + a], u = part[6 * b + 3 + a];
            if (l < s[a][t]) s[a][t] = l;
            if (u > s[3 + a][t]) s[3 + a][t] = u;
        }
    block_box<kBlock>(s);
    if (t == 0) root_cube<kBlock>(s, root);
    __syncthreads();
}

__global__ __launch_bounds__(kBlock) void k_root(const double *part, const int *bad, int nb,
                                                 double box, int *flag, double *root)
{
    __shared__ double s[6][kBlock], rt[4];
    one_root(part, nb, box, s, rt);
    if (threadIdx.x < 4) root[threadIdx.x] = rt[threadIdx.x];
    set_flags(bad, nb, flag);
}

// Several systems' root cubes, a block each: bound by the largest system's chain
// of loads where that is long (a quarter as long with 1024 threads), else by the
// number of blocks (a quarter as many of 1024 at once).  256 / 1024 threads (us): 2^20
// systems of 4 2090 / 9281, 65,536 of 64 136 / 594, 4096 of 500 16 / 43, 700 of 6000 18.7 /
// 22.8, 512 of 8000 18.4 / 19.8, 256 of 15,000 25 / 18, 32 of 65,536 83 / 30; 65,535 of 16
// and one of 10^6 1216 / 643.  The line lies where the largest system has ten
// particles per system of the batch.
constexpr int kSysBlock = 256, kSysBlockWide = 1024, kSysWide = 10;

template <int BS>
__global__ __launch_bounds__(BS) void k_root_sys(const double *x, const int64_t *sys_off,
                                                 const int *bad, int nb, int *flag, double *roots)
{
    __shared__ double s[6][BS];
    const int64_t a = sys_off[blockIdx.x], e = sys_off[blockIdx.x + 1];
    double lo[3], hi[3];
    for (int k = 0; k < 3; ++k) lo[k] = hi[k] = x[3 * a + k];
    for (int64_t p = a + threadIdx.x; p < e; p += BS)
        for (int k = 0; k < 3; ++k) {
            const double v = x[3 * p + k];
            lo[k] = v < lo[k] ? v : lo[k];
            hi[k] = v > hi[k] ? v : hi[k];
        }
    for (int k = 0; k < 3; ++k) {
        s[k][threadIdx.x] = lo[k];
        s[3 + k][threadIdx.x] = hi[k];
    }
    block_box<BS>(s);
    if (threadIdx.x == 0) root_cube<BS>(s, roots + 4 * blockIdx.x);
    if (blockIdx.x == 0) set_flags(bad, nb, flag);
}

// ---- 2. keys ----------------------------------------------------------------

// System of particle p (input or sorted index): off[s] <= p < off[s + 1].
__device__ __forceinline__ int system_of(const int64_t *off, int nsys, int64_t p)
{
    int lo = 0, hi = nsys;
    while (hi - lo > 1) {
        const int mid = (lo + hi) / 2;
        if (off[mid] <= p)
            lo = mid;
        else
            hi = mid;
    }
    return lo;
}

// 63-bit key of a particle: the octant at each depth, below the root cube rt
// (centre, side).
__device__ __forceinline__ uint64_t tree_key(const double *xp, const double *rt)
{
    double c[3] = {rt[0], rt[1], rt[2]};
    double s = rt[3];
    uint64_t k = 0;
    for (int lev = 0; lev < kMaxDepth; ++lev) {
        const double qd = s * 0.25;
        unsigned o = 0;
        for (int a = 0; a < 3; ++a) {
            if (xp[a] >= c[a]) {
                o |= 1u << a;
                c[a] = c[a] + qd;
            } else {
                c[a] = c[a] - qd;
            }
        }
        k = (k << 3) | o;
        s = s * 0.5;
    }
    return k;
}

// roots[4 s .. 4 s + 3] = centre and side of system s's root cube.  The sort
// key is the particle's key or, with lo > 0, its bits from lo up below the
// system's number; and the identity order.
__global__ __launch_bounds__(kBlock) void k_keys(const double *x, int64_t n,
                                                 const int64_t *sys_off, int nsys,
                                                 const double *roots, int lo, uint64_t *key,
                                                 int32_t *idx)
{
    const int64_t p = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (p >= n) return;
    const int sys = nsys > 1 ? system_of(sys_off, nsys, p) : 0;
    const double xp[3] = {x[3 * p], x[3 * p + 1], x[3 * p + 2]};
    const uint64_t k = tree_key(xp, roots + 4 * sys);
    key[p] = lo > 0 ? (uint64_t)sys << (3 * kMaxDepth - lo) | k >> lo : k;
    idx[p] = (int32_t)p;
}

// The keys of one small system; each block finds the root cube itself from
// the checking blocks' boxes, which saves a launch (4 to 5 us), and the first
// also writes it and the flags for the kernels after it.
constexpr int kSmallBoxes = 256;

__global__ __launch_bounds__(kBlock) void k_keys_root(const double *x, int64_t n,
                                                      const double *part, const int *bad, int nb,
                                                      double box, int *flag, double *root,
                                                      uint64_t *key)
{
    __shared__ double s[6][kBlock], rt[4];
    one_root(part, nb, box, s, rt);
    if (blockIdx.x == 0) {
        if (threadIdx.x < 4) root[threadIdx.x] = rt[threadIdx.x];
        set_flags(bad, nb, flag);
    }
    const int64_t p = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (p >= n) return;
    const double xp[3] = {x[3 * p], x[3 * p + 1], x[3 * p + 2]};
    key[p] = tree_key(xp, rt);
}

// ---- 3. cells ----------------------------------------------------------------
//
// All levels at once, from the sorted keys alone.  Two particles lie in one
// cell of depth L iff their keys share L digits, and the sorted particles of a
// cell are consecutive, so with cp(a, b) the number of leading digits that
// the keys of a and b share:
//   * particle k is the first of its cell at depth L iff L > D_k = cp(k - 1, k)
//     (-1 at a system's first particle);
//   * a cell that holds k and w more particles at least has depth at most
//     cp(j, j + w) for a j in [k - w, k], and one of that depth exists.  A cell
//     is split iff it has more than nleaf particles (and depth below 21), so
//     k's leaf has depth LD_k = min(21, 1 + max_j cp(j, j + nleaf)), and k's
//     group, the first cell of at most ncrit particles or a leaf, the depth
//     GD_k that the same formula gives with ncrit.
// Particle k then starts the cells of depths D_k + 1 .. LD_k, and a group iff
// D_k < GD_k; a cell's number is the count of cell starts of lower depth plus
// those of its depth before k: the host's breadth-first ids.  Tiles of
// particles count their starts per depth (k_split), one scan gives every
// tile its first numbers, and k_cells writes the cells: the thread of the
// first particle its geometry and first child, the thread of the first
// particle past it its ends.
// One level per pass, each with two binary searches per octant in the keys,
// a scan and a read by the host, took 0.33 of 1.9 ms on the cube of 2^20
// (now 0.04) and 0.31 ms on a Plummer sphere of 16,384.

// Particles per thread of k_split and k_cells (a tile is a block's particles):
// four share the windows' ends and the scan's entries; up to kSmallTree
// particles one, whose chain is shorter where the blocks do not fill the
// chip (Plummer spheres of 2048 and 16,384: 28 and 31 us for both with four).
constexpr int kPerLarge = 4;
constexpr int64_t kSmallTree = 65536;
// Longest window k_split holds in LDS.  With leaves of more particles (up to
// nleaf) each particle's window is read from memory: a build of 10^6 particles
// takes 11.5 ms at nleaf 5000, 16.3 at 8000 and 88 at 50,000 (1530 and 2750 at
// the first two with a pass per level).
constexpr int kWinMost = 4096;
constexpr int kRows = kMaxDepth + 2;  // depths 0 .. 21 and the groups

// What the build needs of a sorted key array: key(k) = (v[k] & mask) << lo.
struct SortedKeys {
    const uint64_t *v;
    uint64_t mask;
    int lo;
    __device__ __forceinline__ uint64_t operator[](int64_t k) const
    {
        return (v[k] & mask) << lo;
    }
};

__device__ __forceinline__ int common_digits(uint64_t a, uint64_t b)
{
    const uint64_t x = a ^ b;
    return x == 0 ? kMaxDepth : (__builtin_clzll(x) - 1) / 3;
}

// Depths of a particle's start, leaf and group, in one word.
__device__ __forceinline__ int info_d(int32_t v) { return (v & 0xff) - 1; }
__device__ __forceinline__ int info_leaf(int32_t v) { return (v >> 8) & 0xff; }
__device__ __forceinline__ int info_group(int32_t v) { return (v >> 16) & 0xff; }

struct SplitArgs {
    SortedKeys key;
    int64_t n;
    const int64_t *sys_off;  // several systems only
    int nsys, nleaf;
    int ncrit;               // 0: no group row
    int depth;               // digits the sort has ordered
    int rows;                // depth + 1, the group row is row `rows`
    int32_t *info;           // [n] D + 1, LD, GD
    int32_t *count;          // [(rows + 1) nb] starts per depth and tile
    int *deep;               // set if a cell needs more digits
};

// Largest cp(j, j + w) over j in [k - w, k] for the tile's particles k, -1
// if there is none; in LDS bytes a, b of a tile + w each, by doubling: a
// window's maximum is that of two windows half as long.
template <int kTile>
__device__ __forceinline__ const int8_t *window_max(const SplitArgs &A, int64_t k0, int w,
                                                    int8_t *a, int8_t *b, int &half)
{
    const int len = kTile + w;
    int q = A.nsys > 1 ? system_of(A.sys_off, A.nsys, k0 > w ? k0 - w : 0) : 0;
    for (int i = threadIdx.x; i < len; i += kBlock) {
        const int64_t j = k0 - w + i;
        int c = -1;
        if (j >= 0 && j < A.n) {
            int64_t e = A.n;
            if (A.nsys > 1) {
                while (A.sys_off[q + 1] <= j) ++q;
                e = A.sys_off[q + 1];
            }
            if (j + w < e) c = common_digits(A.key[j], A.key[j + w]);
        }
        a[i] = (int8_t)c;
    }
    __syncthreads();
    int p = 1;
    for (; 2 * p <= w + 1; p *= 2) {
        for (int i = threadIdx.x; i < len - p; i += kBlock) b[i] = a[i] > a[i + p] ? a[i] : a[i + p];
        __syncthreads();
        int8_t *s = a;
        a = b;
        b = s;
    }
    half = p;
    return a;
}

template <int kPer>
__global__ __launch_bounds__(kBlock) void k_split(const SplitArgs A, int nb)
{
    constexpr int kTile = kPer * kBlock;
    extern __shared__ int8_t s_win[];
    __shared__ int s_cnt[kBlock / 64][kRows];
    const int t = threadIdx.x;
    const int64_t k0 = (int64_t)blockIdx.x * kTile;
    int leaf[kPer], group[kPer];
    for (int pass = 0; pass < 2; ++pass) {
        const int w = pass ? A.ncrit : A.nleaf;
        if (w <= kWinMost && (!pass || w > 0)) {
            int p;
            __syncthreads();
            const int8_t *m = window_max<kTile>(A, k0, w, s_win, s_win + kTile + w, p);
#pragma unroll
            for (int u = 0; u < kPer; ++u) {
                const int i = t + u * kBlock;
                const int c = m[i] > m[i + w + 1 - p] ? m[i] : m[i + w + 1 - p];
                (pass ? group : leaf)[u] = c;
            }
        } else {
            // a leaf of thousands of particles: the window from memory
#pragma unroll
            for (int u = 0; u < kPer; ++u) {
                const int64_t k = k0 + t + u * kBlock;
                int c = -1;
                if (!pass && k < A.n) {
                    int64_t b = 0, e = A.n;
                    if (A.nsys > 1) {
                        const int q = system_of(A.sys_off, A.nsys, k);
                        b = A.sys_off[q];
                        e = A.sys_off[q + 1];
                    }
                    for (int64_t j = k - w > b ? k - w : b; j <= k && j + w < e; ++j) {
                        const int d = common_digits(A.key[j], A.key[j + w]);
                        c = d > c ? d : c;
                    }
                }
                (pass ? group : leaf)[u] = c;
            }
        }
    }
    int mine = 0;  // lane r: the wave's starts of row r
    const int lane = t & 63;
    bool deep = false;
#pragma unroll
    for (int u = 0; u < kPer; ++u) {
        const int64_t k = k0 + t + u * kBlock;
        int d = kMaxDepth, ld = -1, gd = -1;
        if (k < A.n) {
            ld = leaf[u] + 1 < kMaxDepth ? leaf[u] + 1 : kMaxDepth;
            gd = group[u] + 1 < kMaxDepth ? group[u] + 1 : kMaxDepth;
            deep |= ld > A.depth;
            d = k == 0 ? -1 : common_digits(A.key[k - 1], A.key[k]);
            if (A.nsys > 1 && A.sys_off[system_of(A.sys_off, A.nsys, k)] == k) d = -1;
            A.info[k] = (d + 1) | ld << 8 | gd << 16;
            if (A.ncrit == 0) gd = -1;
        }
        for (int r = 0; r < A.rows; ++r) {
            const int c = (int)__popcll(__ballot(d < r && r <= ld));
            mine += lane == r ? c : 0;
        }
        const int c = (int)__popcll(__ballot(d < gd));
        mine += lane == A.rows ? c : 0;
    }
    if (deep) *A.deep = 1;
    if (lane <= A.rows) s_cnt[t / 64][lane] = mine;
    __syncthreads();
    if (t <= A.rows) {
        int c = 0;
        for (int w = 0; w < kBlock / 64; ++w) c += s_cnt[w][t];
        A.count[(int64_t)t * nb + blockIdx.x] = c;
    }
}

// For the host: table[r] = first number of row r (r <= rows + 1: the cells of
// each depth, then the groups, then the end), after the flags.
__device__ __forceinline__ void write_table(const int32_t *first, int rows, int nb,
                                            const int *flag, int32_t *table)
{
    const int r = threadIdx.x;
    if (r < 4) table[r] = flag[r];
    if (r <= rows + 1) table[4 + r] = first[(int64_t)r * nb];
}

// Exclusive sums of v[0 .. n - 1] to out[0 .. n] in one block (short arrays),
// and the table.
__global__ __launch_bounds__(1024) void k_scan_block(const int32_t *v, int n, int32_t *out,
                                                     int rows, int nb, const int *flag,
                                                     int32_t *table)
{
    typedef hipcub::BlockScan<int, 1024> Scan;
    __shared__ typename Scan::TempStorage tmp;
    int before = 0;
    constexpr int kItems = 4;
    for (int b = 0; b < n; b += 1024 * kItems) {
        int c[kItems], total;
        for (int u = 0; u < kItems; ++u) {
            const int i = b + (int)threadIdx.x * kItems + u;
            c[u] = i < n ? v[i] : 0;
        }
        Scan(tmp).ExclusiveSum(c, c, total);
        for (int u = 0; u < kItems; ++u) {
            const int i = b + (int)threadIdx.x * kItems + u;
            if (i < n) out[i] = before + c[u];
        }
        before += total;
        __syncthreads();
    }
    if (threadIdx.x == 0) out[n] = before;
    __syncthreads();
    write_table(out, rows, nb, flag, table);
}

__global__ void k_table(const int32_t *first, int rows, int nb, const int *flag, int32_t *table)
{
    write_table(first, rows, nb, flag, table);
}

// Several systems: before[q rows + L] = starts of depth L (with those of all
// lower depths) before system q's first particle, q <= nsys.  One wave per
// system, over the particles of its tile.
__global__ __launch_bounds__(64) void k_sys_first(const SplitArgs A, const int32_t *first, int nb,
                                                  int tile, int32_t *before)
{
    const int q = blockIdx.x, lane = threadIdx.x;
    const int64_t e = A.sys_off[q], k0 = e / tile * tile;
    int mine = 0;
    for (int64_t b = k0; b < e; b += 64) {
        const int32_t v = b + lane < e ? A.info[b + lane] : (kMaxDepth + 1);
        for (int r = 0; r < A.rows; ++r) {
            const int c = (int)__popcll(__ballot(info_d(v) < r && r <= info_leaf(v)));
            mine += lane == r ? c : 0;
        }
    }
    if (lane < A.rows)
        before[(int64_t)q * A.rows + lane] = first[(int64_t)lane * nb + k0 / tile] + mine;
}

// cells[q rows + L] = cells of system q at depth L.
__global__ __launch_bounds__(kBlock) void k_sys_cells(const int32_t *before, int64_t n, int rows,
                                                      int32_t *cells)
{
    const int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (i < n) cells[i] = before[i + rows] - before[i];
}

// A batch numbers its cells system by system: shift[q rows + L] takes a
// number in the order of all systems' levels to that one (the exclusive sums
// of the systems' cells less the starts before the system).
__global__ __launch_bounds__(kBlock) void k_sys_shift(const int32_t *before, int64_t n,
                                                      int32_t *shift)
{
    const int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (i < n) shift[i] -= before[i];
}

struct CellArgs {
    SplitArgs s;
    const int32_t *first;  // [(rows + 1) nb + 1] scanned counts
    const int32_t *shift;  // several systems: [nsys rows]
    const double *roots;
    WCell *wc;
    WLink *wl;
    int32_t *parent;       // or NULL
    int32_t *by_level;     // several systems: cells in the order of all levels
    // with a group row: the groups in the layout of the force context, and
    // each one's cell and root cell (several systems)
    int32_t *groups, *groot;
    int64_t *i_off;
    double *gcx, *gcy, *gcz;
    int32_t ngroup0, ng;   // number of the first group start, groups
};

template <int kPer>
__global__ __launch_bounds__(kBlock) void k_cells(const CellArgs C, int nb)
{
    constexpr int kTile = kPer * kBlock;
    constexpr int kChunks = kTile / 64;  // waves' worth of particles per tile
    __shared__ uint64_t s_bal[kChunks][kRows];
    __shared__ int32_t s_pre[kChunks][kRows];
    const SplitArgs &A = C.s;
    const int t = threadIdx.x, lane = t & 63;
    const int64_t k0 = (int64_t)blockIdx.x * kTile;
    int32_t info[kPer];
#pragma unroll
    for (int u = 0; u < kPer; ++u) {
        const int64_t k = k0 + t + u * kBlock;
        info[u] = k < A.n ? A.info[k] : (kMaxDepth + 1);  // past the end: starts nothing
        const int d = info_d(info[u]), ld = info_leaf(info[u]), gd = info_group(info[u]);
        const int c = u * (kBlock / 64) + t / 64;
        for (int r = 0; r < A.rows; ++r) {
            const uint64_t b = __ballot(d < r && r <= ld);
            if (lane == r) s_bal[c][r] = b;
        }
        const uint64_t b = __ballot(d < gd);
        if (lane == A.rows) s_bal[c][lane] = b;
    }
    __syncthreads();
    if (t <= A.rows) {
        int32_t at = C.first[(int64_t)t * nb + blockIdx.x];
        for (int c = 0; c < kChunks; ++c) {
            s_pre[c][t] = at;
            at += (int32_t)__popcll(s_bal[c][t]);
        }
    }
    __syncthreads();
    const uint64_t below = (1ull << lane) - 1ull;
#pragma unroll
    for (int u = 0; u < kPer; ++u) {
        const int64_t k = k0 + t + u * kBlock;
        if (k > A.n) break;
        const int c = u * (kBlock / 64) + t / 64;
        // starts of row r before particle k
        auto before = [&](int r) -> int32_t {
            return s_pre[c][r] + (int32_t)__popcll(s_bal[c][r] & below);
        };
        int q = 0;
        const bool sys_start = k == A.n || info_d(info[u]) < 0;
        if (A.nsys > 1) q = k < A.n ? system_of(A.sys_off, A.nsys, k) : A.nsys;
        const int d = k < A.n ? info_d(info[u]) : -1;
        if (k > 0) {
            // the cells of particle k - 1 that end here
            const int ld = info_leaf(A.info[k - 1]);
            const int32_t *sh =
                C.shift ? C.shift + (int64_t)(q - (sys_start ? 1 : 0)) * A.rows : nullptr;
            for (int l = d + 1; l <= ld; ++l) {
                const int32_t id = before(l) - 1 + (sh ? sh[l] : 0);
                const int32_t ce = l < ld ? before(l + 1) + (sh ? sh[l + 1] : 0) : -1;
                *reinterpret_cast<int2 *>(&C.wl[id].end) = make_int2((int32_t)k, ce);
            }
        }
        if (k == A.n) {
            if (C.groups) C.i_off[C.ng] = k;
            break;
        }
        const int ld = info_leaf(info[u]);
        if (d >= ld) continue;
        const int32_t *sh = C.shift ? C.shift + (int64_t)q * A.rows : nullptr;
        auto number = [&](int l) -> int32_t { return before(l) + (sh ? sh[l] : 0); };
        const uint64_t key = A.key[k];
        const int gd = info_group(info[u]);
        const double *rt = C.roots + 4 * q;
        WCell w;
        w.cx = rt[0];
        w.cy = rt[1];
        w.cz = rt[2];
        w.side = rt[3];
        for (int l = 0; l <= ld; ++l) {
            if (l > 0) {
                const unsigned o = (unsigned)(key >> (3 * (kMaxDepth - l))) & 7u;
                const double qd = w.side * 0.25;
                w.cx = w.cx + ((o & 1u) ? qd : -qd);
                w.cy = w.cy + ((o & 2u) ? qd : -qd);
                w.cz = w.cz + ((o & 4u) ? qd : -qd);
                w.side = w.side * 0.5;
            }
            if (l <= d) continue;
            const int32_t id = number(l);
            double4 *g = reinterpret_cast<double4 *>(C.wc + id);
            *g = make_double4(w.cx, w.cy, w.cz, w.side);
            *reinterpret_cast<int2 *>(&C.wl[id].first) =
                make_int2((int32_t)k, l < ld ? number(l + 1) : -1);
            // at depth d a cell started before k holds it
            if (C.parent)
                C.parent[id] = l == 0 ? -1 : (l - 1 > d ? number(l - 1) : number(l - 1) - 1);
            if (C.by_level) C.by_level[before(l)] = id;
            if (C.groups && l == gd) {
                const int32_t g = before(A.rows) - C.ngroup0;
                C.groups[g] = id;
                C.i_off[g] = k;
                C.gcx[g] = w.cx;
                C.gcy[g] = w.cy;
                C.gcz[g] = w.cz;
                if (C.groot) C.groot[g] = q + sh[0];  // its system's root
            }
        }
    }
}

// Radix sort digit by digit above kRankSortMost (by itself the library merges
// up to 2^20 keys).  A digit of 8 bits costs about 25 us and little more with n
// up to 2^20; the merge sort's passes grow with n and do not depend on the
// bits.  Measured (us, digits / merge), 21 bits: 524,288 88 / 137, 10^6
// 96 / 183; 30 bits: 524,288 115 / 139; 45 bits: 524,288 170 / 144, 10^6
// 181 / 193; 63 bits: 10^6 240 / 199.  So one digit more pays with each
// doubling of n.
typedef rocprim::radix_sort_config<rocprim::default_config, rocprim::default_config,
                                   rocprim::default_config, 0>
    DigitSort;

inline bool sort_by_digits(int64_t n, int bits)
{
    int lg = 0;
    while (((int64_t)2 << lg) <= n) ++lg;
    return (bits + 7) / 8 <= lg - 15;
}

// ---- 4. particles and moments -------------------------------------------------

// Particles in tree order: a leaf's particles are put back in input order (at
// the depth limit they share one key and are in input order already).  One
// thread per sorted particle ranks it in its leaf.
__global__ __launch_bounds__(kBlock) void k_particles_out(const int32_t *sidx,
                                                          const int32_t *info, int64_t n,
                                                          const double *x, const double *m,
                                                          const double *eps2, double eps2_all,
                                                          int32_t *order, PartRec *pool,
                                                          double *xi, double *yi, double *zi,
                                                          double *e2i)
{
    const int64_t k = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (k >= n) return;
    const int32_t p = sidx[k];
    const int32_t v = info[k];
    const int ld = info_leaf(v);
    int64_t at = k;
    if (ld < kMaxDepth) {
        bool start = info_d(v) < ld;
        for (int64_t j = k; !start;) {
            --j;
            at -= sidx[j] > p ? 1 : 0;
            start = info_d(info[j]) < ld;
        }
        for (int64_t j = k + 1; j < n && info_d(info[j]) >= ld; ++j) at += sidx[j] < p ? 1 : 0;
    }
    order[at] = p;
    if (e2i) e2i[at] = eps2 ? eps2[p] : eps2_all;
    PartRec r;
    r.x = x[3 * (int64_t)p];
    r.y = x[3 * (int64_t)p + 1];
    r.z = x[3 * (int64_t)p + 2];
    r.m = m[p];
    pool[at] = r;
    xi[at] = r.x;
    yi[at] = r.y;
    zi[at] = r.z;
}

// Moments of a leaf from its particles, in input order (the host's sums, in
// the host's order): mass and centre of mass, then the traceless
// quadrupole and trace about the centre of mass.  P(k) gives particle k's
// (m, x, y, z).  NMAX > 0: n <= NMAX, and the loops are unrolled to NMAX
// (so that P may index registers); 0: plain loops.
template <int NMAX, typename Part>
__device__ __forceinline__ CellRec leaf_moments(int n, const double ctr[3], Part P)
{
    constexpr int kTrip = NMAX > 0 ? NMAX : 1;
    const int trip = NMAX > 0 ? NMAX : n;
    double M = 0.0, s[3] = {0.0, 0.0, 0.0};
#pragma unroll kTrip
    for (int k = 0; k < trip; ++k) {
        if (k >= n) break;
        const double4 q = P(k);
        M += q.x;
        s[0] += q.x * q.y;
        s[1] += q.x * q.z;
        s[2] += q.x * q.w;
    }
    double cm[3];
    for (int a = 0; a < 3; ++a) cm[a] = M > 0.0 ? s[a] / M : ctr[a];
    double q6[6] = {0, 0, 0, 0, 0, 0}, T = 0.0;
#pragma unroll kTrip
    for (int k = 0; k < trip; ++k) {
        if (k >= n) break;
        const double4 q = P(k);
        const double mp = q.x;
        const double d0 = q.y - cm[0], d1 = q.z - cm[1], d2 = q.w - cm[2];
        const double r2 = d0 * d0 + d1 * d1 + d2 * d2;
        q6[0] += mp * (3.0 * d0 * d0 - r2);
        q6[1] += mp * 3.0 * d0 * d1;
        q6[2] += mp * 3.0 * d0 * d2;
        q6[3] += mp * (3.0 * d1 * d1 - r2);
        q6[4] += mp * 3.0 * d1 * d2;
        q6[5] += mp * (3.0 * d2 * d2 - r2);
        T += mp * r2;
    }
    CellRec r;
    r.x = cm[0];
    r.y = cm[1];
    r.z = cm[2];
    r.m = M;
    r.q00 = q6[0];
    r.q01 = q6[1];
    r.q02 = q6[2];
    r.q11 = q6[3];
    r.q12 = q6[4];
    r.q22 = q6[5];
    r.t = T;
    r.pad = 0.0;
    return r;
}

// One thread per leaf, over its particles in tree order.  A leaf of up to
// kLeafCache particles loads all of them into registers first (independent
// loads, all in flight at once) and sums from there; a larger one (a leaf at
// the depth limit) reads them from memory in each pass.
constexpr int kLeafCache = 8;

__device__ __forceinline__ void store_moments(int32_t c, const CellRec &r, WCell *wc, CellRec *pc)
{
    pc[c] = r;
    wc[c].mx = r.x;
    wc[c].my = r.y;
    wc[c].mz = r.z;
}

__global__ __launch_bounds__(kBlock) void k_moments_leaf(const WLink *wl, int32_t ncell,
                                                         const PartRec *pool, WCell *wc,
                                                         CellRec *pc)
{
    const int32_t c = (int32_t)(blockIdx.x * kBlock + threadIdx.x);
    if (c >= ncell) return;
    const WLink l = wl[c];
    if (l.child0 >= 0) return;
    const int32_t n = l.end - l.first;
    const PartRec *p = pool + l.first;
    const double ctr[3] = {wc[c].cx, wc[c].cy, wc[c].cz};
    auto mem = [&](int k) { return make_double4(p[k].m, p[k].x, p[k].y, p[k].z); };
    if (n <= kLeafCache) {
        double4 q[kLeafCache];
#pragma unroll
        for (int k = 0; k < kLeafCache; ++k)
            if (k < n) q[k] = mem(k);
        store_moments(c, leaf_moments<kLeafCache>(n, ctr, [&](int k) { return q[k]; }), wc, pc);
    } else {
        store_moments(c, leaf_moments<0>(n, ctr, mem), wc, pc);
    }
}

// Moments of an internal cell from its children's, in octant order, by the
// parallel-axis shift: the host's sums in the host's order, with an octet of
// lanes per cell.  Each lane loads one child (contiguous records, all loads in
// flight at once) into LDS, and each sum is one lane's: mass and first
// moments, then the traceless quadrupole and the trace about the centre of
// mass.  With a thread per cell, whose loads followed one another, the depths
// of a Plummer sphere of 16,384 took 75 us (44 now) and those of the
// clustered 2^22 241 us (146).  Leaves stay with a thread each, whose loads
// are all in flight too: with an octet they took 176 us there against 112
// (the octet's second sums do 2.5 times the work).
constexpr int kPart = 11;              // m, x, y, z, six moments, trace
constexpr int kPartStride = kOct + 1;  // (spreads the quantities over banks)
constexpr int kMomOcts = kBlock / kOct;

// The lanes of an octet are in one wave, whose LDS operations complete in
// order: this only keeps the compiler from moving them.
__device__ __forceinline__ void wave_fence()
{
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
}

__device__ __forceinline__ void cell_moments(int32_t c, const WLink &l, double *sh, WCell *wc,
                                             CellRec *pc)
{
    const int k = threadIdx.x % kOct;
    const int n = l.cend - l.child0;
    wave_fence();
    if (k < n) {
        const CellRec &q = pc[l.child0 + k];
        const double v[kPart] = {q.m,   q.x,   q.y,   q.z,   q.q00, q.q01,
                                 q.q02, q.q11, q.q12, q.q22, q.t};
#pragma unroll
        for (int i = 0; i < kPart; ++i) sh[i * kPartStride + k] = v[i];
    }
    wave_fence();
    // lane 0: mass; lanes 1 to 3: first moments (entries past the children
    // are read but not added)
    double sum = 0.0;
#pragma unroll
    for (int i = 0; i < kOct; ++i) {
        const double m = sh[i];
        const double v = sum + (k == 0 ? m : m * sh[(k & 3) * kPartStride + i]);
        sum = i < n ? v : sum;
    }
    const double M = __shfl(sum, 0, kOct);
    const double ctr = k == 1 ? wc[c].cx : (k == 2 ? wc[c].cy : wc[c].cz);
    const double mine = M > 0.0 ? sum / M : ctr;
    const double cm[3] = {__shfl(mine, 1, kOct), __shfl(mine, 2, kOct), __shfl(mine, 3, kOct)};
    // lanes 0 to 5: q00, q01, q02, q11, q12, q22; lane 6: the trace
    const int qa = k < 3 ? 0 : (k < 5 ? 1 : 2), qb = k < 3 ? k : (k < 5 ? k - 2 : 2);
    double q = 0.0;
#pragma unroll
    for (int i = 0; i < kOct; ++i) {
        const double m = sh[i];
        const double d0 = sh[kPartStride + i] - cm[0], d1 = sh[2 * kPartStride + i] - cm[1],
                     d2 = sh[3 * kPartStride + i] - cm[2];
        const double r2 = d0 * d0 + d1 * d1 + d2 * d2;
        const double da = qa == 0 ? d0 : (qa == 1 ? d1 : d2);
        const double db = qb == 0 ? d0 : (qb == 1 ? d1 : d2);
        const double v =
            k >= 6 ? m * r2 : (qa == qb ? m * (3.0 * da * da - r2) : m * 3.0 * da * db);
        const double u = q + (sh[(k < 7 ? 4 + k : 10) * kPartStride + i] + v);
        q = i < n ? u : q;
    }
    double *r = reinterpret_cast<double *>(pc + c);  // x, y, z, m, moments, trace, 0
    r[4 + k] = k < 7 ? q : 0.0;
    if (k < 4) r[(k + 3) & 3] = k == 0 ? M : mine;
    if (k > 0 && k < 4) (&wc[c].mx)[k - 1] = mine;
}

// The internal cells of one depth: numbers lo .. hi - 1, or those of by_level.
__global__ __launch_bounds__(kBlock) void k_moments_level(const WLink *wl, int32_t lo, int32_t hi,
                                                          const int32_t *by_level, WCell *wc,
                                                          CellRec *pc)
{
    __shared__ double sh[kMomOcts][kPart * kPartStride];
    const int64_t i = lo + ((int64_t)blockIdx.x * kBlock + threadIdx.x) / kOct;
    if (i >= hi) return;
    const int32_t c = by_level ? by_level[i] : (int32_t)i;
    const WLink l = wl[c];
    if (l.child0 >= 0) cell_moments(c, l, sh[threadIdx.x / kOct], wc, pc);
}

// The internal cells of depths `top` .. 0, few each, in one block: a launch
// per depth costs more than the work.
struct Depths {
    int32_t first[kMaxDepth + 2];
};
constexpr int kTopCells = 2 * kMomOcts;  // cells of a depth that one block takes

__global__ __launch_bounds__(kBlock) void k_moments_top(const WLink *wl, const Depths D, int top,
                                                        const int32_t *by_level, WCell *wc,
                                                        CellRec *pc)
{
    __shared__ double sh[kMomOcts][kPart * kPartStride];
    const int o = threadIdx.x / kOct;
    for (int d = top; d >= 0; --d) {
        for (int32_t i = D.first[d] + o; i < D.first[d + 1]; i += kMomOcts) {
            const int32_t c = by_level ? by_level[i] : i;
            const WLink l = wl[c];
            if (l.child0 >= 0) cell_moments(c, l, sh[o], wc, pc);
        }
        __syncthreads();
    }
}

// ---- 5. groups ----------------------------------------------------------------

__global__ __launch_bounds__(kBlock) void k_fill_i32(int32_t *v, int64_t n, int32_t val)
{
    const int64_t k = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (k < n) v[k] = val;
}

// Groups of more particles than k_split's windows span: a cell is a group iff
// it has at most ncrit particles or is a leaf, and its parent (if any) has
// more than ncrit.  gstart[first] = cell id.
__global__ __launch_bounds__(kBlock) void k_group_mark(const WLink *wl, const int32_t *parent,
                                                       int32_t ncell, int ncrit, int32_t *gstart)
{
    const int32_t c = (int32_t)(blockIdx.x * kBlock + threadIdx.x);
    if (c >= ncell) return;
    const WLink l = wl[c];
    const bool cond = l.end - l.first <= ncrit || l.child0 < 0;
    const int32_t p = parent[c];
    const bool top = p < 0 || wl[p].end - wl[p].first > ncrit;
    if (cond && top) gstart[l.first] = c;
}

struct NonNegative {
    __host__ __device__ bool operator()(const int32_t &v) const { return v >= 0; }
};

// The same from the groups' cells (groups that k_cells did not find): their
// layout in the force context, and each group's root cell (the number of its
// system's root: shift[q rows] + q; several systems only).
__global__ __launch_bounds__(kBlock) void k_groups_out(const WCell *wc, const WLink *wl,
                                                       const int32_t *groups, int64_t ng,
                                                       int64_t n, const int64_t *sys_off,
                                                       int nsys, const int32_t *shift, int rows,
                                                       int64_t *i_off, double *gcx, double *gcy,
                                                       double *gcz, int32_t *groot)
{
    const int64_t g = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (g > ng) return;
    if (g == ng) {
        i_off[ng] = n;
        return;
    }
    const int32_t c = groups[g], f = wl[c].first;
    i_off[g] = f;
    gcx[g] = wc[c].cx;
    gcy[g] = wc[c].cy;
    gcz[g] = wc[c].cz;
    if (groot) {
        const int q = system_of(sys_off, nsys, f);
        groot[g] = q + shift[(int64_t)q * rows];
    }
}

// ---- 6. walk -----------------------------------------------------------------

// |v - box rint(v / box)|, the distance to the nearest periodic image (|v|
// without a box).  For |v| < box / 4 the quotient rounds to below 1/2, rint
// gives 0 and the result is |v|: the division, a long instruction sequence
// in FP64, is taken only for the far cells.
__device__ __forceinline__ double abs_min_image(double v, double box)
{
    const double a = ::fabs(v);
    if (box > 0.0 && !(a < 0.25 * box)) return ::fabs(v - box * ::rint(v / box));
    return a;
}

// Whether the cell holds the group: no smaller than it, and its particles
// include the group's (cells of one depth are disjoint, so the cell is then
// the group's ancestor at that depth, or the group).
__device__ __forceinline__ bool contains(const WCell &C, const WLink &L, const WCell &G,
                                         const WLink &GL)
{
    return C.side >= G.side && L.first <= GL.first && L.end >= GL.end;
}

struct WalkArgs {
    const int32_t *groups;
    const int32_t *groot;              // root cell of each group's tree (NULL: 0)
    int64_t ng;
    const WCell *wc;
    const WLink *wl;
    double theta2, rcut, box;
    double rdrop2;                     // accepted cells this far (squared) from the
                                       // box of the group's particles are beyond the
                                       // cutoff for all of them and left out; 0: no
                                       // cutoff
    int64_t *jp_cnt, *jc_cnt;          // count pass
    const int64_t *jp_off, *jc_off;    // fill pass
    int32_t *jp_idx, *jc_idx;
    int *flag;                         // set if a stack (1) or the level walk's
                                       // octets (2) would overflow
    int *most;                         // most cells that a group opens
    int64_t cap_p, cap_c;              // slot sizes of the one-walk mode
    int frames;                        // frame stack depth: levels of the tree
    const double *gbox;                // [6 ng] lo, hi of each group's particles
                                       // (with a cutoff)
};

// A child of an opened cell, as the walk classifies it, in two ints:
//   skipped (beyond the cutoff)         {-1, 0}
//   j-cell id                           {id, 0}
//   particles first .. first + count-1  {first, count}, count >= 1 (an
//                                        accepted one-particle cell or an
//                                        opened leaf)
//   opened internal cell                {-2 - child0, nchild}
// CUT: with a cutoff or a periodic box.
template <bool CUT>
__device__ __forceinline__ int2 classify(const WalkArgs &W, int32_t id, const WCell &G,
                                         const WLink &GL, const double *gb)
{
    const WCell C = W.wc[id];
    const WLink L = W.wl[id];
    const double box = CUT ? W.box : 0.0;
    const double gc[3] = {G.cx, G.cy, G.cz};
    if (!contains(C, L, G, GL)) {
        if (CUT && W.rcut > 0.0) {
            const double cc[3] = {C.cx, C.cy, C.cz};
            double d2 = 0.0;
            for (int k = 0; k < 3; ++k) {
                const double v = ::fmax(abs_min_image(cc[k] - gc[k], box) -
                                            0.5 * (C.side + G.side), 0.0);
                d2 += v * v;
            }
            if (d2 > W.rcut * W.rcut) return make_int2(-1, 0);
        }
        const double cm[3] = {C.mx, C.my, C.mz};
        double d2 = 0.0;
        for (int k = 0; k < 3; ++k) {
            const double v = ::fmax(abs_min_image(cm[k] - gc[k], box) - 0.5 * G.side, 0.0);
            d2 += v * v;
        }
        if (C.side * C.side < W.theta2 * d2) {
            // beyond the cutoff for every particle of the group
            if (CUT && W.rdrop2 > 0.0) {
                // distance to the box of the group's particles (centre
                // gb[0..2], half widths gb[3..5])
                double b2 = 0.0;
                for (int k = 0; k < 3; ++k) {
                    const double v = ::fmax(abs_min_image(cm[k] - gb[k], box) - gb[3 + k], 0.0);
                    b2 += v * v;
                }
                if (b2 >= W.rdrop2) return make_int2(-1, 0);
            }
            return L.end - L.first == 1 ? make_int2(L.first, 1) : make_int2(id, 0);
        }
    }
    if (L.child0 < 0) return make_int2(L.first, L.end - L.first);
    return make_int2(-2 - L.child0, L.cend - L.child0);
}

// Data movement inside an octet (8 aligned lanes) by DPP, on the VALU:
// an inclusive prefix sum and a sum returned to every lane.  DPP works in
// rows of 16 lanes, which hold two octets; every read below stays inside
// the reading lane's octet (row_shr by d is used only by lanes k >= d).
template <int CTRL>
__device__ __forceinline__ int dpp(int v)
{
    return __builtin_amdgcn_update_dpp(0, v, CTRL, 0xf, 0xf, false);
}

// Exclusive prefix sum; m: per distance 1, 2, 4 all ones in the lanes that
// have a lane of their octet so far below (k >= 1, 2, 4), else zero.
__device__ __forceinline__ int octet_scan(int v, const int *m)
{
    const int own = v;
    v += __builtin_amdgcn_update_dpp(0, v, 0x111, 0xf, 0xf, true) & m[0];  // row_shr:1
    v += __builtin_amdgcn_update_dpp(0, v, 0x112, 0xf, 0xf, true) & m[1];  // row_shr:2
    v += __builtin_amdgcn_update_dpp(0, v, 0x114, 0xf, 0xf, true) & m[2];  // row_shr:4
    return v - own;
}

__device__ __forceinline__ int octet_sum(int v)
{
    v += dpp<0x141>(v);  // row_half_mirror: lane 7 - k of the octet
    v += dpp<0xB1>(v);   // quad_perm [1, 0, 3, 2]: lane k ^ 1
    v += dpp<0x4E>(v);   // quad_perm [2, 3, 0, 1]: lane k ^ 2
    return v;
}

// dst[0 .. n - 1] = first, first + 1, ...  A leaf's run is a few entries at any
// alignment, and its lane's stores each touch a line of their own: four
// entries per store.
struct alignas(4) Ids4 {
    int32_t v[4];
};

__device__ __forceinline__ void put_run(int32_t *dst, int32_t first, int32_t n)
{
    int32_t j = 0;
    for (; j + 4 <= n; j += 4)
        *reinterpret_cast<Ids4 *>(dst + j) = {{first + j, first + j + 1, first + j + 2,
                                               first + j + 3}};
    for (; j < n; ++j) dst[j] = first + j;
}

// Centre and half widths of the box (lo, hi) of group gi's particles, with
// the host builder's operations (zero without a cutoff).
__device__ __forceinline__ void group_box(const WalkArgs &W, int64_t gi, double gb[6])
{
    for (int k = 0; k < 6; ++k) gb[k] = 0.0;
    if (W.rdrop2 > 0.0)
        for (int k = 0; k < 3; ++k) {
            const double lo = W.gbox[6 * gi + k], hi = W.gbox[6 * gi + 3 + k];
            gb[k] = 0.5 * (lo + hi);
            gb[3 + k] = 0.5 * (hi - lo);
        }
}

// Walk modes: count the entries; fill the lists at exact offsets; or fill
// fixed slots of cap_p / cap_c entries per group and count (one walk).
enum WalkMode { kWalkCount = 0, kWalkFill = 1, kWalkSlots = 2 };

// Level walk: a block of NW waves walks one group breadth first.  Every
// opened cell is an octet of lanes, one per child; all cells that a level
// opens are classified together, so the chain of dependent loads is as long
// as the tree is deep (the octet walk's is one per opened cell, some
// hundreds).  Then two passes over the octets give every entry its place in
// the depth-first, octant order: totals from the deepest level up, positions
// from the root down.  Octets are numbered as they come up (LDS counter),
// those opened by one octet in a row; the lists do not depend on the numbers.
// LDS keeps 16 B per octet, so that occupancy is not bound by it: the first
// child's id, the number of the first octet opened (16 bits) over the
// children's kinds (2 bits each), and the totals (summed by one lane per
// octet), replaced by the octet's position on the way down.  `cap` octets fit:
// a group that opens more sets *W.flag = 2 (its other cells are left out) and
// the host walks again with the octet walk.
// A rebuild's walk took 0.75 ms on the cube of 10^6, 4.6 on the 2^24 lattice
// at ncrit 128 and 0.65 on a Plummer sphere of 16,384 (989 groups, each a
// chain of about 200 openings) with the octet walk, and 0.20, 3.3 and 0.042
// with this one; with the totals by a lane per octet, four entries per store
// of a run and no cutoff terms without a cutoff 0.18, 3.15 and 0.040 (1.30 ->
// 1.11 on 256 systems, 1.36 -> 1.24 on the clustered 2^22).
// What is left is the classification's arithmetic (VALU busy 88 % of the time
// on the lattice, 71 % on the cube) and one chain of loads per level on small
// inputs.  Keeping the children as classified (72 B per octet) left two blocks
// per CU on inputs with a few long groups: the clustered 2^22 walk was slower
// than the octet walk.
constexpr uint32_t kNodeNone = 0, kNodeCell = 1, kNodeRun = 2, kNodeOpen = 3;

template <int MODE, int NW, bool CUT>
__global__ __launch_bounds__(64 * NW) void k_walk_level(const WalkArgs W, int cap)
{
    extern __shared__ int2 s_walk[];
    int2 *s_sum = s_walk;                                // {cells, particles}
    int32_t *s_c0 = reinterpret_cast<int32_t *>(s_walk + cap);
    uint32_t *s_kind = reinterpret_cast<uint32_t *>(s_c0 + cap);  // first: nchild
    __shared__ int s_lev[kFrames + 1];
    __shared__ int s_cnt;
    const int t = threadIdx.x;
    const int k = t & (kOct - 1);
    const int o = t / kOct;
    const unsigned per = gridDim.x / kXcds;  // as in k_walk
    const int64_t gi = (int64_t)(blockIdx.x % kXcds) * per + blockIdx.x / kXcds;
    if (gi >= W.ng) return;
    const int32_t gid = W.groups[gi];
    const WCell G = W.wc[gid];
    const WLink GL = W.wl[gid];
    double gb[6];
    group_box(W, gi, gb);
    int64_t pb = 0, cb = 0, pe = 0, ce = 0;  // where this group's entries go
    if (MODE == kWalkFill) {
        pb = W.jp_off[gi];
        cb = W.jc_off[gi];
        pe = W.jp_off[gi + 1];
        ce = W.jc_off[gi + 1];
    } else if (MODE == kWalkSlots) {
        pb = gi * W.cap_p;
        cb = gi * W.cap_c;
        pe = pb + W.cap_p;
        ce = cb + W.cap_c;
    }
    const WLink R = W.wl[W.groot ? W.groot[gi] : 0];
    if (R.child0 < 0) {
        // a one-leaf tree: the root contains the group and is opened
        if (MODE != kWalkCount)
            for (int32_t j = t; j < R.end - R.first && pb + j < pe; j += 64 * NW)
                W.jp_idx[pb + j] = R.first + j;
        if (MODE != kWalkFill && t == 0) {
            W.jp_cnt[gi] = R.end - R.first;
            W.jc_cnt[gi] = 0;
        }
        return;
    }
    if (t == 0) {
        s_c0[0] = R.child0;
        s_kind[0] = (uint32_t)children(R);
        s_cnt = 1;
    }
    __syncthreads();
    int lo = 0, hi = 1, nl = 0;
    bool full = false;
    while (hi > lo) {
        if (t == 0) s_lev[nl] = lo;
        for (int q = lo + o; q < hi; q += kOct * NW) {
            const int32_t c0 = s_c0[q];
            const int2 e = k < (int)s_kind[q] ? classify<CUT>(W, c0 + k, G, GL, gb)
                                              : make_int2(-1, 0);
            bool open = e.x <= -2;
            const uint64_t bal = __ballot(open);
            int ch = 0;  // octet of this lane's (opened) child, or the next one's
            if (bal != 0) {
                const int first = __builtin_ctzll(bal);
                int base = 0;
                if ((t & 63) == first) base = atomicAdd(&s_cnt, (int)__popcll(bal));
                base = __builtin_amdgcn_readlane(base, first);
                ch = base + (int)__builtin_amdgcn_mbcnt_hi(
                                (uint32_t)(bal >> 32),
                                __builtin_amdgcn_mbcnt_lo((uint32_t)bal, 0u));
                if (open) {
                    if (ch < cap) {
                        s_c0[ch] = -2 - e.x;
                        s_kind[ch] = (uint32_t)e.y;
                    } else {
                        full = true;
                        open = false;
                    }
                }
            }
            const bool cell = e.x >= 0 && e.y == 0, run = e.x >= 0 && e.y > 0;
            const uint32_t kind =
                (cell ? kNodeCell : run ? kNodeRun : open ? kNodeOpen : kNodeNone) << (2 * k);
            const int own = octet_sum(run ? e.y : 0);
            const uint32_t kinds = (uint32_t)octet_sum((int)kind);
            if (k == 0) {
                s_kind[q] = kinds | (uint32_t)ch << 16;
                s_sum[q].y = own;
            }
        }
        __syncthreads();
        lo = hi;
        hi = s_cnt < cap ? s_cnt : cap;
        ++nl;
        __syncthreads();
    }
    if (t == 0) s_lev[nl] = hi;
    if (full) *W.flag = 2;
    __syncthreads();
    // totals, one lane per octet over the octets it opened
    for (int l = nl - 1; l >= 0; --l) {
        const int b = s_lev[l], f = s_lev[l + 1];
        for (int q = b + t; q < f; q += 64 * NW) {
            const uint32_t kinds = s_kind[q], up = kinds >> 1;
            int2 v = make_int2(__popc(kinds & ~up & 0x5555u), s_sum[q].y);
            const int c = (int)(kinds >> 16), e = c + __popc(kinds & up & 0x5555u);
            for (int j = c; j < e; ++j) {
                const int2 u = s_sum[j];
                v.x += u.x;
                v.y += u.y;
            }
            s_sum[q] = v;
        }
        __syncthreads();
    }
    if (t == 0) {
        if (MODE != kWalkFill) {
            W.jc_cnt[gi] = s_sum[0].x;
            W.jp_cnt[gi] = s_sum[0].y;
            // most cells opened by a group (its octets), for the next
            // build's LDS (the plain read spares most groups the atomic)
            if (*(volatile int *)W.most < hi) atomicMax(W.most, hi);
        }
        s_sum[0] = make_int2(0, 0);
    }
    if (MODE == kWalkCount) return;
    __syncthreads();
    // entries left in the group's segments; a slot overflow is detected from
    // the counts
    const int cleft = (int)(ce - cb < INT_MAX ? ce - cb : INT_MAX);
    const int pleft = (int)(pe - pb < INT_MAX ? pe - pb : INT_MAX);
    int32_t *const jc = W.jc_idx + cb, *const jp = W.jp_idx + pb;
    const int below[3] = {k >= 1 ? -1 : 0, k >= 2 ? -1 : 0, k >= 4 ? -1 : 0};
    const uint32_t lower = 0x5555u & ((1u << (2 * k)) - 1u);
    for (int l = 0; l < nl; ++l) {
        const int b = s_lev[l], f = s_lev[l + 1];
        for (int q = b + o; q < f; q += kOct * NW) {
            const int2 at = s_sum[q];
            const uint32_t kinds = s_kind[q], kind = (kinds >> (2 * k)) & 3u;
            const int32_t id = s_c0[q] + k;
            int32_t first = 0;
            int2 v = make_int2(kind == kNodeCell ? 1 : 0, 0);
            int ch = 0;
            if (kind == kNodeOpen) {
                // its number among those that the octet opened
                ch = (int)(kinds >> 16) + __popc(kinds & (kinds >> 1) & lower);
                v = s_sum[ch];
            } else if (kind == kNodeRun) {
                const WLink L = W.wl[id];
                first = L.first;
                v.y = L.end - L.first;
            }
            const int c0 = at.x + octet_scan(v.x, below);
            const int p0 = at.y + octet_scan(v.y, below);
            if (kind == kNodeOpen) {
                s_sum[ch] = make_int2(c0, p0);
            } else if (kind == kNodeCell) {
                if (c0 < cleft) jc[c0] = id;
            } else if (kind == kNodeRun) {
                put_run(jp + p0, first, pleft - p0 < v.y ? pleft - p0 : v.y);
            }
        }
        __syncthreads();
    }
}

// Octet walk: the 8 lanes of an octet walk one group.  Opening an internal
// cell loads and classifies all of its children at once, one per lane, and
// pushes them as a frame; a frame is emitted in octant order up to its next
// opened internal child, whose subtree is walked before the rest of the
// frame.  The lists therefore come out in the depth-first, octant order of
// the host builder's walk, while the chain of dependent loads per group is
// one per opened cell instead of one per visited cell.  The current frame
// lives in registers; each lane keeps its child's entry of every frame in
// LDS for the return from a subtree, and the frame's child count and cursor
// are stored once per octet, written by all 8 lanes with the same value.
// Control flow is uniform within an octet.  The fill pass writes only
// inside the group's own segments of the lists.  Its memory is bounded by
// the tree's depth alone: it takes the groups that open more cells than the
// level walk's LDS holds.
template <int MODE>
__global__ __launch_bounds__(kWalkBlock) void k_walk(const WalkArgs W)
{
    // frame stack, W.frames deep (the tree's depth): a child entry per lane,
    // then nchild | cursor << 8 per octet (dynamic LDS: a shallow tree
    // leaves room for more resident waves)
    extern __shared__ int2 s_walk[];
    int2 (*s_ent)[kWalkBlock] = reinterpret_cast<int2 (*)[kWalkBlock]>(s_walk);
    int32_t (*s_hdr)[kWalkBlock / kOct] = reinterpret_cast<int32_t (*)[kWalkBlock / kOct]>(
        s_walk + (size_t)W.frames * kWalkBlock);
    const int t = threadIdx.x;
    const int k = t & (kOct - 1);
    const int o = t / kOct;
    // The hardware hands blocks to the XCDs round robin; XCD x walks the
    // contiguous range of groups [x per, (x + 1) per) of blocks, so that
    // neighbouring groups, whose walks read the same cells, share an L2.
    const unsigned per = gridDim.x / kXcds;
    const unsigned lb = (blockIdx.x % kXcds) * per + blockIdx.x / kXcds;
    const int64_t gi = (int64_t)lb * (kWalkBlock / kOct) + o;
    if (gi >= W.ng) return;  // whole octets leave; no block-wide synchronisation below
    const int32_t gid = W.groups[gi];
    const WCell G = W.wc[gid];
    const WLink GL = W.wl[gid];
    double gb[6];
    group_box(W, gi, gb);
    int64_t np = 0, nc = 0;
    constexpr bool FILL = MODE != kWalkCount;
    int64_t pb = 0, cb = 0, pe = 0, ce = 0;  // where this group's entries go
    if (MODE == kWalkFill) {
        pb = W.jp_off[gi];
        cb = W.jc_off[gi];
        pe = W.jp_off[gi + 1];
        ce = W.jc_off[gi + 1];
    } else if (MODE == kWalkSlots) {
        pb = gi * W.cap_p;
        cb = gi * W.cap_c;
        pe = pb + W.cap_p;
        ce = cb + W.cap_c;
    }
    const WLink R = W.wl[W.groot ? W.groot[gi] : 0];
    const int below[3] = {k >= 1 ? -1 : 0, k >= 2 ? -1 : 0, k >= 4 ? -1 : 0};
    int sp = 0, nch = 0, cur = 0, opened = 0;
    int2 e = make_int2(-1, 0);
    if (R.child0 < 0) {
        // a one-leaf tree: the root contains the group and is opened
        if (FILL)
            for (int32_t j = k; j < R.end - R.first && pb + j < pe; j += kOct)
                W.jp_idx[pb + j] = R.first + j;
        np = R.end - R.first;
    } else {
        nch = children(R);
        e = k < nch ? classify<true>(W, R.child0 + k, G, GL, gb) : make_int2(-1, 0);
        s_ent[0][t] = e;
        sp = 1;
        opened = 1;
    }
    // Each round: emit and return from frames (cheap) until the octet must
    // open a child or is done, then open it (loads and classification).
    // Octets of a wave reach their next opening at different steps; taking
    // the openings in a round of their own lets the expensive part run for
    // all octets of the wave together.
    while (sp > 0) {
        int32_t c0 = 0;
        int n2 = -1;  // >= 0: open the cell whose children are c0 .. c0 + n2 - 1
        for (;;) {
            const bool mine = k >= cur && k < nch;
            // the first opened internal child at or after the cursor
            const uint64_t bal = __ballot(mine && e.x <= -2);
            const uint32_t om = (uint32_t)(bal >> (t & 63 & ~(kOct - 1))) & 0xffu;
            const int kstar = om ? __builtin_ctz(om) : nch;
            // emit the children before it
            const bool em = mine && k < kstar && e.x >= 0;
            const int vp = em ? e.y : 0;            // particles
            const int vc = em && e.y == 0 ? 1 : 0;  // cells
            if (FILL) {
                const int ip = octet_scan(vp, below), ic = octet_scan(vc, below);
                if (em) {
                    if (e.y == 0) {
                        const int64_t q = cb + nc + ic;
                        if (q < ce) W.jc_idx[q] = e.x;
                    } else {
                        // the entries that fit in the group's segment (none
                        // past it: a slot overflow is detected from the counts)
                        const int64_t q = pb + np + ip;
                        put_run(W.jp_idx + q, e.x,
                                (int32_t)(pe - q < (int64_t)e.y ? pe - q : e.y));
                    }
                }
            }
            np += octet_sum(vp);
            nc += octet_sum(vc);
            if (kstar < nch) {
                // descend into child kstar; this frame resumes after it
                c0 = -2 - __shfl(e.x, kstar, kOct);
                const int n = __shfl(e.y, kstar, kOct);
                cur = kstar + 1;
                if (sp < W.frames) {
                    s_hdr[sp - 1][o] = nch | cur << 8;
                    n2 = n;
                    break;
                }
                if (k == 0) *W.flag = 1;  // the subtree is left out; the build fails
                continue;
            }
            if (--sp == 0) break;
            e = s_ent[sp - 1][t];
            const int hdr = s_hdr[sp - 1][o];
            nch = hdr & 0xff;
            cur = hdr >> 8;
        }
        if (n2 < 0) break;
        e = k < n2 ? classify<true>(W, c0 + k, G, GL, gb) : make_int2(-1, 0);
        s_ent[sp][t] = e;
        nch = n2;
        cur = 0;
        ++sp;
        ++opened;
    }
    if (MODE != kWalkFill && k == 0) {
        W.jp_cnt[gi] = np;
        W.jc_cnt[gi] = nc;
        if (*(volatile int *)W.most < opened) atomicMax(W.most, opened);  // as in k_walk_level
    }
}

// Bounding box (lo[3], hi[3]) of each group's particles, for the cutoff
// drop; an octet of lanes per group over its particles in tree order
// (minimum and maximum do not depend on the order).
__global__ __launch_bounds__(kBlock) void k_group_box(const WLink *wl, const int32_t *groups,
                                                      int64_t ng, const double *x, const double *y,
                                                      const double *z, double *gbox)
{
    const int64_t g = ((int64_t)blockIdx.x * kBlock + threadIdx.x) / kOct;
    const int k = threadIdx.x % kOct;
    if (g >= ng) return;
    const WLink l = wl[groups[g]];
    const double *xs[3] = {x, y, z};
    double lo[3], hi[3];
    for (int a = 0; a < 3; ++a) {
        lo[a] = __builtin_inf();
        hi[a] = -__builtin_inf();
    }
    for (int32_t p = l.first + k; p < l.end; p += kOct)
        for (int a = 0; a < 3; ++a) {
            const double v = xs[a][p];
            lo[a] = v < lo[a] ? v : lo[a];
            hi[a] = v > hi[a] ? v : hi[a];
        }
    for (int a = 0; a < 3; ++a) {
        for (int h = kOct / 2; h > 0; h /= 2) {
            const double u = __shfl_xor(lo[a], h, kOct), v = __shfl_xor(hi[a], h, kOct);
            lo[a] = u < lo[a] ? u : lo[a];
            hi[a] = v > hi[a] ? v : hi[a];
        }
        if (k == 0) {
            gbox[6 * g + a] = lo[a];
            gbox[6 * g + 3 + a] = hi[a];
        }
    }
}

// Lists of one-walk builds: group g's entries [0, off[g+1] - off[g]) of
// its slot (cap entries from g cap) to out[off[g] ...]; one wave per group.
__global__ __launch_bounds__(kBlock) void k_compact(int64_t ng, const int64_t *off,
                                                    const int32_t *slot, int64_t cap,
                                                    int32_t *out)
{
    const int64_t g = (int64_t)blockIdx.x * (kBlock / 64) + threadIdx.x / 64;
    if (g >= ng) return;
    const int lane = threadIdx.x & 63;
    const int64_t o = off[g], n = off[g + 1] - o;
    const int32_t *src = slot + g * cap;
    for (int64_t j = lane; j < n; j += 64) out[o + j] = src[j];
}

}  // namespace

hipError_t launch_compact_lists(int64_t ng, const int64_t *off, const int32_t *slot,
                                int64_t cap, int32_t *out, hipStream_t s)
{
    if (ng <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_compact, dim3(blocks(ng, kBlock / 64)), dim3(kBlock), 0, s, ng, off,
                       slot, cap, out);
    return hipGetLastError();
}

// ---- host orchestration ---------------------------------------------------------

int build_tree_lists(const TreeParams &P, TreeOut &O, hipStream_t s, std::string *err)
{
    DevArray *B = O.buf;
    const int64_t n = P.n;
    int code = BHQ_OK;
    const char *what = "";
    auto hip = [&](hipError_t e, const char *w) -> bool {
        if (e == hipSuccess) return true;
        code = (e == hipErrorOutOfMemory || e == hipErrorMemoryAllocation) ? BHQ_E_NOMEM
                                                                            : BHQ_E_HIP;
        what = w;
        return false;
    };
    auto fail = [&]() -> int {
        if (err) {
            *err = std::string("device list build: ") + what;
            if (code == BHQ_E_HIP || code == BHQ_E_NOMEM)
                *err += std::string(" (") + hipGetErrorString(hipGetLastError()) + ")";
        }
        return code;
    };
#define STEP(expr, w)              \
    do {                           \
        if (!hip((expr), (w))) return fail(); \
    } while (0)
#define LAUNCHED(w) STEP(hipGetLastError(), w)

    // input check, systems, root cubes
    const int nsys = (int)P.nsys;
    STEP(B[T_FLAG].reserve(kFlags * 4), "allocation");
    int *flag = B[T_FLAG].as<int>();  // non-finite, softening, too deep; the walk's from 4
    STEP(B[T_ROOTS].reserve((size_t)nsys * 4 * sizeof(double)), "allocation");
    double *roots = B[T_ROOTS].as<double>();
    const int64_t *sys_off = nullptr;
    std::vector<int32_t> so32;  // read by the copy below until the synchronisation
    const bool one = nsys == 1 && n <= kRankSortMost;  // the keys' kernel finds the root
    int nbox = 0;
    double *part = nullptr;
    int *bad = nullptr;
    {
        nbox = (int)std::min<int64_t>(one ? kSmallBoxes : kBboxBlocks, blocks(n, kBlock));
        STEP(B[T_BBOX].reserve((size_t)nbox * (6 * sizeof(double) + sizeof(int))), "allocation");
        part = B[T_BBOX].as<double>();
        bad = reinterpret_cast<int *>(part + (size_t)nbox * 6);
        hipLaunchKernelGGL(k_check, dim3(nbox), dim3(kBlock), 0, s, P.x, P.m, P.eps2, n, bad,
                           nsys == 1 && !(P.box > 0.0) ? part : nullptr);
        LAUNCHED("finite check");
        if (nsys == 1 && !one) {
            hipLaunchKernelGGL(k_root, dim3(1), dim3(kBlock), 0, s, part, bad, nbox, P.box, flag,
                               roots);
            LAUNCHED("root cube");
        } else if (nsys > 1) {
            STEP(B[T_SYSOFF].reserve((size_t)(nsys + 1) * 8), "allocation");
            STEP(B[T_SYSOFF32].reserve((size_t)(nsys + 1) * 4), "allocation");
            STEP(hipMemcpyAsync(B[T_SYSOFF].p, P.sys_off, (size_t)(nsys + 1) * 8,
                                hipMemcpyHostToDevice, s),
                 "copy");
            so32.resize((size_t)nsys + 1);
            int64_t largest = 0;
            for (int q = 0; q < nsys; ++q) {
                so32[(size_t)q] = (int32_t)P.sys_off[q];
                largest = std::max(largest, P.sys_off[q + 1] - P.sys_off[q]);
            }
            so32[(size_t)nsys] = (int32_t)P.sys_off[nsys];
            STEP(hipMemcpyAsync(B[T_SYSOFF32].p, so32.data(), (size_t)(nsys + 1) * 4,
                                hipMemcpyHostToDevice, s),
                 "copy");
            sys_off = B[T_SYSOFF].as<int64_t>();
            if (largest > kSysWide * P.nsys)
                hipLaunchKernelGGL(k_root_sys<kSysBlockWide>, dim3((unsigned)nsys),
                                   dim3(kSysBlockWide), 0, s, P.x, sys_off, bad, nbox, flag,
                                   roots);
            else
                hipLaunchKernelGGL(k_root_sys<kSysBlock>, dim3((unsigned)nsys), dim3(kSysBlock),
                                   0, s, P.x, sys_off, bad, nbox, flag, roots);
            LAUNCHED("root cubes");
        }
    }

    // keys, sort, cells per depth
    STEP(B[T_KEY].reserve((size_t)n * 8), "allocation");
    STEP(B[T_KEY2].reserve((size_t)n * 8), "allocation");
    STEP(B[T_IDX0].reserve((size_t)n * 4), "allocation");
    STEP(B[T_IDX1].reserve((size_t)n * 4), "allocation");
    STEP(B[T_INFO].reserve((size_t)n * 4), "allocation");
    int sysbits = 0;
    while (((int64_t)1 << sysbits) < nsys) ++sysbits;
    // Stable sort of (key, input index) on key bits [lo, 63).  A tree of L
    // levels (depths below L) reads L - 1 digits of the keys, so it needs the
    // bits from 3 (kMaxDepth + 1 - L) up; the order inside a leaf does not
    // matter (its particles are put back in input order).  A rebuild sorts the
    // bits its previous depth needs; if the tree turns out deeper, the keys
    // are sorted again on all bits.  The systems of a batch are sorted in one
    // go where system and key bits fit 64, else as segments.
    bool joint = false;
    auto sort_keys = [&](int lo) -> bool {
        uint64_t *k0 = B[T_KEY].as<uint64_t>(), *k1 = B[T_KEY2].as<uint64_t>();
        int32_t *i0 = B[T_IDX0].as<int32_t>(), *i1 = B[T_IDX1].as<int32_t>();
        const int32_t *so = B[T_SYSOFF32].as<int32_t>();
        joint = nsys > 1 && lo > 0 && 3 * kMaxDepth - lo + sysbits <= 64;
        const int b0 = joint ? 0 : lo, b1 = joint ? 3 * kMaxDepth - lo + sysbits : 3 * kMaxDepth;
        // (a key's 21 levels are too much arithmetic for the few blocks that
        // sort the tiles: formed there they cost 5 to 9 us more)
        if (one)
            hipLaunchKernelGGL(k_keys_root, dim3(blocks(n, kBlock)), dim3(kBlock), 0, s, P.x, n,
                               part, bad, nbox, P.box, flag, roots, k0);
        else
            hipLaunchKernelGGL(k_keys, dim3(blocks(n, kBlock)), dim3(kBlock), 0, s, P.x, n,
                               sys_off, nsys, roots, joint ? lo : 0, k0, i0);
        if (!hip(hipGetLastError(), "keys")) return false;
        if ((nsys == 1 || joint) && n <= kRankSortMost && b1 < 64)
            return hip(rank_sort(StoredKeys<uint64_t>{k0}, n, b0, b1, k0, i0, k1, i1, s), "sort");
        auto run = [&](void *tmp, size_t &bytes) -> hipError_t {
            if ((nsys == 1 || joint) && sort_by_digits(n, b1 - b0))
                return rocprim::radix_sort_pairs<DigitSort>(tmp, bytes, k0, k1, i0, i1,
                                                            (unsigned)n, (unsigned)b0,
                                                            (unsigned)b1, s);
            if (nsys == 1 || joint)
                return hipcub::DeviceRadixSort::SortPairs(tmp, bytes, k0, k1, i0, i1, (int)n, b0,
                                                          b1, s);
            return hipcub::DeviceSegmentedRadixSort::SortPairs(tmp, bytes, k0, k1, i0, i1, (int)n,
                                                               nsys, so, so + 1, b0, b1, s);
        };
        size_t tmp = 0;
        if (!hip(run(nullptr, tmp), "sort size")) return false;
        if (!hip(B[T_SORT].reserve(std::max(tmp, B[T_SORT].cap)), "allocation")) return false;
        return hip(run(B[T_SORT].p, tmp), "sort");
    };
    const bool small = n <= kSmallTree;
    const int tile = (small ? 1 : kPerLarge) * kBlock;
    const int nb = (int)blocks(n + 1, tile);
    const bool group_row = P.ncrit <= kWinMost;
    volatile int32_t *table = static_cast<int32_t *>(O.host);
    static_assert(4 + kRows + 2 <= 64, "level table");
    int lo = P.spec_levels > 0 ? 3 * (kMaxDepth + 1 - std::max(2, P.spec_levels)) : 0;
    SplitArgs S{};
    int rows = 0;
    for (;;) {
        if (!sort_keys(lo)) return fail();
        S.key = joint ? SortedKeys{B[T_KEY2].as<uint64_t>(),
                                   ((uint64_t)1 << (3 * kMaxDepth - lo)) - 1, lo}
                      : SortedKeys{B[T_KEY2].as<uint64_t>(), ~(uint64_t)0, 0};
        S.n = n;
        S.sys_off = sys_off;
        S.nsys = nsys;
        S.nleaf = P.nleaf;
        S.ncrit = group_row ? P.ncrit : 0;
        S.depth = kMaxDepth - lo / 3;
        S.rows = rows = S.depth + 1;
        S.info = B[T_INFO].as<int32_t>();
        const int ncount = (rows + 1) * nb;
        STEP(B[T_NCH].reserve((size_t)(ncount + 1) * 4), "allocation");
        STEP(B[T_NOFF].reserve((size_t)(ncount + 1) * 4), "allocation");
        S.count = B[T_NCH].as<int32_t>();
        S.deep = flag + 2;
        const int win = std::max(P.nleaf <= kWinMost ? P.nleaf : 0, S.ncrit);
        const size_t lds = 2 * (size_t)(tile + win);
        if (small)
            hipLaunchKernelGGL(k_split<1>, dim3((unsigned)nb), dim3(kBlock), lds, s, S, nb);
        else
            hipLaunchKernelGGL(k_split<kPerLarge>, dim3((unsigned)nb), dim3(kBlock), lds, s, S,
                               nb);
        LAUNCHED("cell starts");
        if (ncount <= 16384) {
            hipLaunchKernelGGL(k_scan_block, dim3(1), dim3(1024), 0, s, S.count, ncount,
                               B[T_NOFF].as<int32_t>(), rows, nb, flag,
                               static_cast<int32_t *>(O.host));
            LAUNCHED("scan");
        } else {
            size_t st = 0;
            STEP(hipcub::DeviceScan::ExclusiveSum(nullptr, st, S.count, B[T_NOFF].as<int32_t>(),
                                                  ncount + 1, s),
                 "scan size");
            STEP(B[T_SORT].reserve(std::max(st, B[T_SORT].cap)), "allocation");
            STEP(hipcub::DeviceScan::ExclusiveSum(B[T_SORT].p, st, S.count,
                                                  B[T_NOFF].as<int32_t>(), ncount + 1, s),
                 "scan");
            hipLaunchKernelGGL(k_table, dim3(1), dim3(64), 0, s, B[T_NOFF].as<int32_t>(), rows,
                               nb, flag, static_cast<int32_t *>(O.host));
            LAUNCHED("level table");
        }
        STEP(hipStreamSynchronize(s), "sync");
        if (table[0]) {
            code = BHQ_E_NONFINITE;
            what = "non-finite position or mass";
            return fail();
        }
        if (table[1]) {
            code = BHQ_E_ARG;
            what = "eps2 must be finite and >= 2^-126";
            return fail();
        }
        if (!table[2] || lo == 0) break;
        lo = 0;
        STEP(hipMemsetAsync(flag + 2, 0, 4, s), "memset");
    }
    Depths level{};  // depth l is cells [first[l], first[l + 1]) (in level order)
    int nlevels = 0;
    for (int l = 0; l < rows; ++l) {
        level.first[l] = table[4 + l];
        level.first[l + 1] = table[4 + l + 1];
        if (table[4 + l + 1] < table[4 + l]) {
            code = BHQ_E_RANGE;
            what = "more than 2^31 cells";
            return fail();
        }
        if (table[4 + l + 1] > table[4 + l]) nlevels = l + 1;
    }
    const int32_t ncell = table[4 + rows];

    // cells
    STEP(B[T_WC].reserve((size_t)ncell * sizeof(WCell)), "allocation");
    STEP(B[T_WL].reserve((size_t)ncell * sizeof(WLink)), "allocation");
    WCell *wc = B[T_WC].as<WCell>();
    WLink *wl = B[T_WL].as<WLink>();
    CellArgs CA{};
    CA.s = S;
    CA.first = B[T_NOFF].as<int32_t>();
    CA.roots = roots;
    CA.wc = wc;
    CA.wl = wl;
    CA.ngroup0 = ncell;
    if (nsys > 1) {
        // each system's cells in a row
        const int64_t tab = (int64_t)nsys * rows;
        STEP(B[T_LSC].reserve((size_t)(tab + rows) * 4), "allocation");
        STEP(B[T_LSN].reserve((size_t)tab * 4), "allocation");
        STEP(B[T_SHIFT].reserve((size_t)tab * 4), "allocation");
        STEP(B[T_BYLEVEL].reserve((size_t)ncell * 4), "allocation");
        int32_t *before = B[T_LSC].as<int32_t>(), *cnt = B[T_LSN].as<int32_t>();
        int32_t *shift = B[T_SHIFT].as<int32_t>();
        hipLaunchKernelGGL(k_sys_first, dim3((unsigned)nsys + 1), dim3(64), 0, s, S, CA.first, nb,
                           tile, before);
        LAUNCHED("system cells");
        hipLaunchKernelGGL(k_sys_cells, dim3(blocks(tab, kBlock)), dim3(kBlock), 0, s, before, tab,
                           rows, cnt);
        LAUNCHED("system cells");
        size_t st = 0;
        STEP(hipcub::DeviceScan::ExclusiveSum(nullptr, st, cnt, shift, (int)tab, s), "scan size");
        STEP(B[T_SORT].reserve(std::max(st, B[T_SORT].cap)), "allocation");
        STEP(hipcub::DeviceScan::ExclusiveSum(B[T_SORT].p, st, cnt, shift, (int)tab, s), "scan");
        hipLaunchKernelGGL(k_sys_shift, dim3(blocks(tab, kBlock)), dim3(kBlock), 0, s, before, tab,
                           shift);
        LAUNCHED("system cells");
        CA.shift = shift;
        CA.by_level = B[T_BYLEVEL].as<int32_t>();
    }
    int64_t ng = group_row ? table[4 + rows + 1] - ncell : 0;
    STEP(B[T_GROUPS].reserve((size_t)(group_row ? ng : n) * 4), "allocation");
    int32_t *groups = B[T_GROUPS].as<int32_t>();
    auto group_arrays = [&]() -> bool {
        return hip(O.i_off->reserve((size_t)(ng + 1) * 8), "allocation") &&
               hip(O.gcx->reserve((size_t)ng * 8), "allocation") &&
               hip(O.gcy->reserve((size_t)ng * 8), "allocation") &&
               hip(O.gcz->reserve((size_t)ng * 8), "allocation") &&
               (nsys == 1 || hip(B[T_GROOT].reserve((size_t)ng * 4), "allocation"));
    };
    if (group_row) {
        if (!group_arrays()) return fail();
        CA.groups = groups;
        CA.groot = nsys > 1 ? B[T_GROOT].as<int32_t>() : nullptr;
        CA.i_off = O.i_off->as<int64_t>();
        CA.gcx = O.gcx->as<double>();
        CA.gcy = O.gcy->as<double>();
        CA.gcz = O.gcz->as<double>();
        CA.ng = (int32_t)ng;
    } else {
        STEP(B[T_PARENT].reserve((size_t)ncell * 4), "allocation");
        CA.parent = B[T_PARENT].as<int32_t>();
    }
    if (small)
        hipLaunchKernelGGL(k_cells<1>, dim3((unsigned)nb), dim3(kBlock), 0, s, CA, nb);
    else
        hipLaunchKernelGGL(k_cells<kPerLarge>, dim3((unsigned)nb), dim3(kBlock), 0, s, CA, nb);
    LAUNCHED("cells");

    // particles in tree order, in the layout of the force context
    STEP(O.order->reserve((size_t)n * 4), "allocation");
    STEP(O.pool_p->reserve((size_t)n * sizeof(PartRec)), "allocation");
    STEP(O.xi->reserve((size_t)n * 8), "allocation");
    STEP(O.yi->reserve((size_t)n * 8), "allocation");
    STEP(O.zi->reserve((size_t)n * 8), "allocation");
    const bool soft = P.eps2 || P.eps2_all > 0.0;
    if (soft) STEP(O.e2i->reserve((size_t)n * 8), "allocation");
    hipLaunchKernelGGL(k_particles_out, dim3(blocks(n, kBlock)), dim3(kBlock), 0, s,
                       B[T_IDX1].as<int32_t>(), S.info, n, P.x, P.m, P.eps2, P.eps2_all,
                       O.order->as<int32_t>(), O.pool_p->as<PartRec>(), O.xi->as<double>(),
                       O.yi->as<double>(), O.zi->as<double>(),
                       soft ? O.e2i->as<double>() : nullptr);
    LAUNCHED("particle pool");

    // moments straight into the cell pool (the deepest cells are leaves)
    STEP(O.pool_c->reserve((size_t)ncell * sizeof(CellRec)), "allocation");
    CellRec *pc = O.pool_c->as<CellRec>();
    hipLaunchKernelGGL(k_moments_leaf, dim3(blocks(ncell, kBlock)), dim3(kBlock), 0, s, wl, ncell,
                       O.pool_p->as<PartRec>(), wc, pc);
    LAUNCHED("leaf moments");
    int top = -1;
    while (top + 1 <= nlevels - 2 &&
           level.first[top + 2] - level.first[top + 1] <= kTopCells)
        ++top;
    for (int l = nlevels - 2; l > top; --l) {
        const int32_t b = level.first[l], e = level.first[l + 1];
        hipLaunchKernelGGL(k_moments_level, dim3(blocks((int64_t)(e - b) * kOct, kBlock)),
                           dim3(kBlock), 0, s, wl, b, e, CA.by_level, wc, pc);
        LAUNCHED("cell moments");
    }
    if (top >= 0) {
        hipLaunchKernelGGL(k_moments_top, dim3(1), dim3(kBlock), 0, s, wl, level, top, CA.by_level,
                           wc, pc);
        LAUNCHED("cell moments");
    }

    if (!group_row) {
        // groups in depth-first order
        STEP(B[T_GSTART].reserve((size_t)n * 4), "allocation");
        STEP(B[T_NSEL].reserve(64), "allocation");
        hipLaunchKernelGGL(k_fill_i32, dim3(blocks(n, kBlock)), dim3(kBlock), 0, s,
                           B[T_GSTART].as<int32_t>(), n, -1);
        LAUNCHED("fill");
        hipLaunchKernelGGL(k_group_mark, dim3(blocks(ncell, kBlock)), dim3(kBlock), 0, s, wl,
                           CA.parent, ncell, P.ncrit, B[T_GSTART].as<int32_t>());
        LAUNCHED("groups");
        size_t st = 0;
        STEP(hipcub::DeviceSelect::If(nullptr, st, B[T_GSTART].as<int32_t>(), groups,
                                      B[T_NSEL].as<int32_t>(), (int)n, NonNegative(), s),
             "select size");
        STEP(B[T_SORT].reserve(std::max(st, B[T_SORT].cap)), "allocation");
        STEP(hipcub::DeviceSelect::If(B[T_SORT].p, st, B[T_GSTART].as<int32_t>(), groups,
                                      B[T_NSEL].as<int32_t>(), (int)n, NonNegative(), s),
             "select");
        int32_t ng32 = 0;
        STEP(hipMemcpyAsync(&ng32, B[T_NSEL].p, 4, hipMemcpyDeviceToHost, s), "copy");
        STEP(hipStreamSynchronize(s), "sync");
        ng = ng32;
        if (!group_arrays()) return fail();
        hipLaunchKernelGGL(k_groups_out, dim3(blocks(ng + 1, kBlock)), dim3(kBlock), 0, s, wc, wl,
                           groups, ng, n, sys_off, nsys, CA.shift, rows, O.i_off->as<int64_t>(),
                           O.gcx->as<double>(), O.gcy->as<double>(), O.gcz->as<double>(),
                           nsys > 1 ? B[T_GROOT].as<int32_t>() : nullptr);
        LAUNCHED("groups");
    }

    // walk: count, offsets, fill
    STEP(B[T_JPCNT].reserve((size_t)(ng + 1) * 8), "allocation");
    STEP(B[T_JCCNT].reserve((size_t)(ng + 1) * 8), "allocation");
    STEP(O.jp_off->reserve((size_t)(ng + 1) * 8), "allocation");
    STEP(O.jc_off->reserve((size_t)(ng + 1) * 8), "allocation");
    WalkArgs W{};
    W.groups = groups;
    W.groot = nsys > 1 ? B[T_GROOT].as<int32_t>() : nullptr;
    W.ng = ng;
    W.wc = wc;
    W.wl = wl;
    W.theta2 = P.theta * P.theta;
    W.rcut = P.rcut;
    {
        const double r = P.rcut * (1.0 + 0x1p-16);
        W.rdrop2 = P.rcut > 0.0 ? r * r : 0.0;
    }
    W.box = P.box;
    W.jp_cnt = B[T_JPCNT].as<int64_t>();
    W.jc_cnt = B[T_JCCNT].as<int64_t>();
    W.flag = flag + 4;
    W.most = W.flag + 2;
    // one frame per level below the root: enough for the deepest opened cell
    W.frames = std::max(1, std::min(kFrames, nlevels));
    const size_t walk_lds = (size_t)W.frames * (kWalkBlock * sizeof(int2) + kWalkBlock / kOct * 4);
    // octets the level walk's LDS holds; 0: octet walk
    int oct_cap = std::min(std::max(P.cap_o, 0), kOctMost);
    // Waves per group of the level walk: two, or four when there are too few
    // groups to fill the chip (2048: 16 waves per CU either way), where the
    // time is the chain of one group.  With one, two and four waves a rebuild's
    // walk took 80, - and 42 us (Plummer sphere of 16,384, 989 groups), and
    // force evaluations 15.2, 13.8 and 14.2 ms (clustered 2^22, whose longest
    // groups end last with one wave) and TreePM steps 31.0, 31.1 and 32.3 ms
    // (2^24 lattice).
    const bool wide = ng <= 2048;
    auto walk = [&](int mode) -> bool {
        if (oct_cap > 0) {
            const size_t lds = (size_t)oct_cap * kOctBytes;
            const dim3 g((unsigned)((ng + kXcds - 1) / kXcds * kXcds));
            const bool cut = W.rcut > 0.0 || W.box > 0.0;
            auto launch = [&](auto two, auto four, auto two_cut, auto four_cut) {
                if (wide)
                    hipLaunchKernelGGL(cut ? four_cut : four, g, dim3(256), lds, s, W, oct_cap);
                else
                    hipLaunchKernelGGL(cut ? two_cut : two, g, dim3(128), lds, s, W, oct_cap);
            };
#define BHQ_WALKS(mode)                                                   \
    launch(k_walk_level<mode, 2, false>, k_walk_level<mode, 4, false>,    \
           k_walk_level<mode, 2, true>, k_walk_level<mode, 4, true>)
            if (mode == kWalkCount)
                BHQ_WALKS(kWalkCount);
            else if (mode == kWalkFill)
                BHQ_WALKS(kWalkFill);
            else
                BHQ_WALKS(kWalkSlots);
#undef BHQ_WALKS
        } else {
            const dim3 g(walk_blocks(ng)), b(kWalkBlock);
            if (mode == kWalkCount)
                hipLaunchKernelGGL(k_walk<kWalkCount>, g, b, walk_lds, s, W);
            else if (mode == kWalkFill)
                hipLaunchKernelGGL(k_walk<kWalkFill>, g, b, walk_lds, s, W);
            else
                hipLaunchKernelGGL(k_walk<kWalkSlots>, g, b, walk_lds, s, W);
        }
        return hip(hipGetLastError(), "walk");
    };
    W.gbox = nullptr;
    if (W.rdrop2 > 0.0) {
        STEP(B[T_GBOX].reserve((size_t)ng * 6 * 8), "allocation");
        hipLaunchKernelGGL(k_group_box, dim3(blocks(ng * kOct, kBlock)), dim3(kBlock), 0, s, wl,
                           groups, ng, O.xi->as<double>(), O.yi->as<double>(),
                           O.zi->as<double>(), B[T_GBOX].as<double>());
        LAUNCHED("group boxes");
        W.gbox = B[T_GBOX].as<double>();
    }
    // One walk into fixed slots when the caller gives capacities (from an
    // earlier build) and the slots fit the memory bound; else count first.
    const bool slots = P.cap_p > 0 && P.cap_c > 0 &&
                       (double)ng * (double)(P.cap_p + P.cap_c) * 4.0 <= (double)P.slot_bytes;
    if (slots) {
        STEP(B[T_JPSLOT].reserve((size_t)ng * (size_t)P.cap_p * 4), "allocation");
        STEP(B[T_JCSLOT].reserve((size_t)ng * (size_t)P.cap_c * 4), "allocation");
        W.cap_p = P.cap_p;
        W.cap_c = P.cap_c;
        W.jp_idx = B[T_JPSLOT].as<int32_t>();
        W.jc_idx = B[T_JCSLOT].as<int32_t>();
    }
    // offsets, dispatch order, and what the host needs of them, with the walk
    ListPlan L;
    L.ng = ng;
    L.i_off = O.i_off->as<int64_t>();
    L.jp_cnt = W.jp_cnt;
    L.jc_cnt = W.jc_cnt;
    L.jp_off = O.jp_off->as<int64_t>();
    L.jc_off = O.jc_off->as<int64_t>();
    L.window = P.window;
    L.tail = P.tail;
    L.xcds = P.xcds;
    L.flag = W.flag;
    L.stats = reinterpret_cast<int64_t *>(static_cast<char *>(O.host) + kBuildStats);
    L.order = P.window > 0 ? O.slots : nullptr;
    L.scratch = O.scratch;
    volatile int64_t *stats = L.stats;
    for (;;) {
        if (!walk(slots ? kWalkSlots : kWalkCount)) return fail();
        code = plan_lists_launch(L, s, err);
        if (code != BHQ_OK) return code;
        STEP(hipStreamSynchronize(s), "sync");
        if (stats[kStatWalk] != 2) break;
        // a group opened more cells than the level walk's LDS holds
        oct_cap = 0;
        STEP(hipMemsetAsync(W.flag, 0, 16, s), "memset");
    }
    if (stats[kStatWalk]) {
        code = BHQ_E_RANGE;
        what = "walk stack overflow";
        return fail();
    }
    if (L.order) {
        code = plan_lists_finish(L, s, err);
        if (code != BHQ_OK) return code;
        O.nslots = stats[kStatSlots];
    }
    const int64_t most = stats[kStatOpened];
    const int64_t njp = stats[kStatParts], njc = stats[kStatCells];
    const int64_t max_p = stats[kStatMaxParts], max_c = stats[kStatMaxCells];
    O.one_walk = slots && max_p <= P.cap_p && max_c <= P.cap_c;
    O.slot_p = O.slot_c = 0;
    if (O.one_walk) {
        // every group's entries are in its slot: the slots become the lists
        // (the force kernel reads group g from g * slot size), and the old
        // list arrays the slots of the next rebuild
        std::swap(*O.jp_idx, B[T_JPSLOT]);
        std::swap(*O.jc_idx, B[T_JCSLOT]);
        O.slot_p = P.cap_p;
        O.slot_c = P.cap_c;
    } else {
        // The list arrays trade places with the slots on the next one-walk
        // rebuild, so they are given the size of its slots where those will
        // be used: then neither needs to grow again.
        int64_t want_p = njp, want_c = njc;
        const int64_t np2 = next_slot_cap(P.cap_p, max_p), nc2 = next_slot_cap(P.cap_c, max_c);
        if ((double)ng * (double)(np2 + nc2) * 4.0 <= (double)slot_memory_bound(njp, njc)) {
            want_p = std::max(want_p, ng * np2);
            want_c = std::max(want_c, ng * nc2);
        }
        STEP(O.jp_idx->reserve((size_t)std::max<int64_t>(want_p, 1) * 4), "allocation");
        STEP(O.jc_idx->reserve((size_t)std::max<int64_t>(want_c, 1) * 4), "allocation");
        W.jp_off = O.jp_off->as<int64_t>();
        W.jc_off = O.jc_off->as<int64_t>();
        W.jp_idx = O.jp_idx->as<int32_t>();
        W.jc_idx = O.jc_idx->as<int32_t>();
        if (oct_cap > 0) oct_cap = std::max(1, (int)most);
        if (!walk(kWalkFill)) return fail();
        STEP(hipStreamSynchronize(s), "sync");
    }
    O.max_o = most;
    O.max_p = max_p;
    O.max_c = max_c;

    O.ng = ng;
    O.njp = njp;
    O.njc = njc;
    O.ncell = ncell;
    O.nlevels = nlevels;
#undef STEP
#undef LAUNCHED
    return BHQ_OK;
}

}  // namespace bhq
