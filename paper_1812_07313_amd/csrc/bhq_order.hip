// bhq_order.hip -- the XCD dispatch order (launch slot table) computed on
// the GPU for lists that are already in device memory.  The steps and the
// arithmetic are those of the host planner (plan_order in bhq_api.cpp):
//   cost c_g = ni_g (100 njp_g + 265 njc_g + 100), in 64-bit integers;
//   B_g = sum of c_h over h < g (exact prefix sums), T = B_ng;
//   piece x_g = floor((2 B_g + c_g) / (2 T) * xcds), in FP64 with the same
//   operations, clamped to [0, xcds - 1]: contiguous pieces of equal cost;
//   in each piece, windows of `window` consecutive groups and one window of
//   its last `tail` groups, each sorted by cost, largest first (ties in
//   group order);
//   slot b of the table holds entry b / xcds of piece b % xcds, or -1.
// So the table is the host planner's, entry for entry.
//
// The same passes turn the walk's list lengths into offsets and reduce what
// the host needs (totals, longest lists, slots), so that a build waits for
// them once: with library scans and reductions, a read of the pieces by the
// host and an upload of the windows, these steps took 13 launches and four
// synchronisations (about 110 us of a 2048-particle build).
#include <hip/hip_runtime.h>
#include <hipcub/hipcub.hpp>

#include <algorithm>

#include "bhq.h"
#include "bhq_internal.h"

namespace bhq {

namespace {

constexpr int kBlock = 256;
constexpr int kItems = 8;
constexpr int kTile = kBlock * kItems;  // groups per block of the sums
constexpr int kSortMax = 1024;          // largest window sorted by one block
constexpr int kMaxXcds = 64;

// Sums over groups of the list entries, the cost and the shapes' work, and
// the largest of each.
constexpr int kTerms = 3 + kShapes;
struct Sums {
    uint64_t sum[kTerms], most[kTerms];
};

struct PlanArgs {
    int64_t ng;
    const int64_t *i_off;
    const int64_t *jp_cnt, *jc_cnt;  // list lengths, or NULL: from the offsets
    int64_t *jp_off, *jc_off;        // written if lengths are given
    int window, tail, xcds;
    Sums *tile;                      // [tiles] each tile's sums, then the sums
                                     // before it; [tiles] the totals
    uint64_t *cost;                  // [ng]
    int64_t *start;                  // [xcds + 1] first group of each piece
    int32_t *order;
    int64_t cap;                     // entries of order
    const int *flag;                 // the walk's, or NULL
    int64_t *stats;
};

// Entries and cost of group g (0 past the end).
__device__ __forceinline__ void group_terms(const PlanArgs &A, int64_t g, uint64_t (&v)[3])
{
    v[0] = v[1] = v[2] = 0;
    if (g >= A.ng) return;
    v[0] = (uint64_t)(A.jp_cnt ? A.jp_cnt[g] : A.jp_off[g + 1] - A.jp_off[g]);
    v[1] = (uint64_t)(A.jc_cnt ? A.jc_cnt[g] : A.jc_off[g + 1] - A.jc_off[g]);
    v[2] = order_cost(A.i_off[g + 1] - A.i_off[g], (int64_t)v[0], (int64_t)v[1]);
}

// Adds a group's terms, the shapes' work among them.
__device__ __forceinline__ void add_group(const PlanArgs &A, int64_t g, Sums &s)
{
    uint64_t e[3], v[kTerms];
    group_terms(A, g, e);
    if (g >= A.ng) return;
    const uint64_t entries = list_cost((int64_t)e[0], (int64_t)e[1]);
    for (int k = 0; k < 3; ++k) v[k] = e[k];
    for (int q = 0; q < kShapes; ++q)
        v[3 + q] = entries * shape_lanes(A.i_off[g + 1] - A.i_off[g], q);
    for (int k = 0; k < kTerms; ++k) {
        s.sum[k] += v[k];
        s.most[k] = v[k] > s.most[k] ? v[k] : s.most[k];
    }
}

// Sums of s.sum and the largest of s.most over the block's threads, to all of
// them.
__device__ __forceinline__ void block_reduce(Sums &s)
{
    __shared__ Sums wave[kBlock / 64];
    for (int h = 32; h > 0; h /= 2)
        for (int k = 0; k < kTerms; ++k) {
            s.sum[k] += __shfl_xor((unsigned long long)s.sum[k], h);
            const uint64_t m = __shfl_xor((unsigned long long)s.most[k], h);
            s.most[k] = m > s.most[k] ? m : s.most[k];
        }
    if (threadIdx.x % 64 == 0) wave[threadIdx.x / 64] = s;
    __syncthreads();
    s = wave[0];
    for (int w = 1; w < kBlock / 64; ++w)
        for (int k = 0; k < kTerms; ++k) {
            s.sum[k] += wave[w].sum[k];
            s.most[k] = wave[w].most[k] > s.most[k] ? wave[w].most[k] : s.most[k];
        }
}

__global__ __launch_bounds__(kBlock) void k_tile_sums(const PlanArgs A)
{
    Sums s{};
    for (int u = 0; u < kItems; ++u)
        add_group(A, (int64_t)blockIdx.x * kTile + u * kBlock + threadIdx.x, s);
    block_reduce(s);
    if (threadIdx.x == 0) A.tile[blockIdx.x] = s;
}

// Exclusive sums of the tiles' entries and costs (in sum[0..2]), totals after
// them; one block.
__global__ __launch_bounds__(kBlock) void k_tile_scan(const PlanArgs A, int tiles)
{
    typedef hipcub::BlockScan<uint64_t, kBlock> Scan;
    __shared__ typename Scan::TempStorage tmp;
    uint64_t at[3] = {0, 0, 0};
    Sums all{};
    for (int b = 0; b < tiles; b += kBlock) {
        const int i = b + (int)threadIdx.x;
        const Sums t = i < tiles ? A.tile[i] : Sums{};
        for (int k = 0; k < 3; ++k) {
            uint64_t ex, tot;
            Scan(tmp).ExclusiveSum(t.sum[k], ex, tot);
            __syncthreads();
            if (i < tiles) A.tile[i].sum[k] = at[k] + ex;
            at[k] += tot;
        }
        for (int k = 0; k < kTerms; ++k) {
            all.sum[k] += t.sum[k];
            all.most[k] = t.most[k] > all.most[k] ? t.most[k] : all.most[k];
        }
    }
    block_reduce(all);
    if (threadIdx.x == 0) A.tile[tiles] = all;
}

__device__ __forceinline__ void write_work(const PlanArgs &A, const Sums &s)
{
    for (int q = 0; q < kShapes; ++q) {
        A.stats[kStatWork + q] = (int64_t)s.sum[3 + q];
        A.stats[kStatMaxWork + q] = (int64_t)s.most[3 + q];
    }
}

// A tile's offsets, costs and pieces; the statistics.  ONE: the only tile,
// whose sums are the block's own; a second block has the shapes' work (2 us more
// in the first).
template <bool ONE>
__global__ __launch_bounds__(kBlock) void k_offsets(const PlanArgs A, int tiles)
{
    typedef hipcub::BlockScan<uint64_t, kBlock> Scan;
    typedef hipcub::BlockReduce<uint64_t, kBlock> Reduce;
    __shared__ union {
        typename Scan::TempStorage scan;
        typename Reduce::TempStorage reduce;
    } tmp;
    if constexpr (ONE) {
        if (blockIdx.x == 1) {
            Sums s{};
            for (int64_t g = threadIdx.x; g < A.ng; g += kBlock) add_group(A, g, s);
            block_reduce(s);
            if (threadIdx.x == 0) write_work(A, s);
            return;
        }
    }
    const int64_t g0 = (int64_t)blockIdx.x * kTile + (int64_t)threadIdx.x * kItems;
    uint64_t v[3][kItems], cost[kItems], mx[3] = {0, 0, 0};
    for (int u = 0; u < kItems; ++u) {
        uint64_t x[3];
        group_terms(A, g0 + u, x);
        for (int k = 0; k < 3; ++k) {
            v[k][u] = x[k];
            mx[k] = x[k] > mx[k] ? x[k] : mx[k];
        }
        cost[u] = x[2];
    }
    Sums all{};
    uint64_t before[3] = {0, 0, 0};
    for (int k = 0; k < 3; ++k) {
        Scan(tmp.scan).ExclusiveSum(v[k], v[k], all.sum[k]);
        __syncthreads();
    }
    if constexpr (ONE) {
        for (int k = 0; k < 3; ++k) {
            all.most[k] = Reduce(tmp.reduce).Reduce(mx[k], hipcub::Max());  // (thread 0)
            __syncthreads();
        }
    } else {
        for (int k = 0; k < 3; ++k) before[k] = A.tile[blockIdx.x].sum[k];
        all = A.tile[tiles];
    }
    // the piece of the group before this thread's first: its cost interval
    // ends where the first's begins
    int xp = -1;
    if (g0 > 0 && g0 < A.ng) {
        uint64_t x[3];
        group_terms(A, g0 - 1, x);
        xp = order_piece(before[2] + v[2][0] - x[2], x[2], all.sum[2], A.xcds, g0 - 1, A.ng);
    }
    for (int u = 0; u < kItems; ++u) {
        const int64_t g = g0 + u;
        if (g >= A.ng) break;
        if (A.jp_cnt) {
            A.jp_off[g] = (int64_t)(before[0] + v[0][u]);
            A.jc_off[g] = (int64_t)(before[1] + v[1][u]);
        }
        A.cost[g] = cost[u];
        const int x = order_piece(before[2] + v[2][u], cost[u], all.sum[2], A.xcds, g, A.ng);
        for (int p = xp + 1; p <= x; ++p) A.start[p] = g;
        xp = x;
        if (g == A.ng - 1) {
            for (int p = x + 1; p <= A.xcds; ++p) A.start[p] = A.ng;
            if (A.jp_cnt) {
                A.jp_off[A.ng] = (int64_t)all.sum[0];
                A.jc_off[A.ng] = (int64_t)all.sum[1];
            }
        }
    }
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        A.stats[kStatParts] = (int64_t)all.sum[0];
        A.stats[kStatCells] = (int64_t)all.sum[1];
        A.stats[kStatMaxParts] = (int64_t)all.most[0];
        A.stats[kStatMaxCells] = (int64_t)all.most[1];
        A.stats[kStatCost] = (int64_t)all.sum[2];
        A.stats[kStatMaxCost] = (int64_t)all.most[2];
        if (!ONE) write_work(A, all);
        A.stats[kStatWalk] = A.flag ? A.flag[0] : 0;
        A.stats[kStatOpened] = A.flag ? A.flag[2] : 0;
    }
}

// a before b in a window: larger cost, then smaller group index
__device__ __forceinline__ bool costlier(uint64_t ca, int32_t ga, uint64_t cb, int32_t gb)
{
    return ca > cb || (ca == cb && ga < gb);
}

// One block per window, found from the pieces: piece p has windows of
// `window` groups from its start and one (perhaps empty) of its last `tail`
// groups.  Bitonic sort with one group per thread: partners less than a wave
// apart exchange by shuffles, others through LDS (ten of the 55 exchanges
// of a tail of 1024; with LDS and a barrier for each, and 256 threads, the
// cube's windows took 46 us, now 13).  The last window of a piece also marks
// its empty slots.
__global__ __launch_bounds__(kSortMax) void k_window_sort(const PlanArgs A)
{
    __shared__ uint64_t sc[kSortMax];
    __shared__ int32_t sg[kSortMax];
    const int t = threadIdx.x;
    int64_t longest = 0;
    for (int p = 0; p < A.xcds; ++p) {
        const int64_t k = A.start[p + 1] - A.start[p];
        longest = k > longest ? k : longest;
    }
    if (blockIdx.x == 0 && t == 0) A.stats[kStatSlots] = longest * A.xcds;
    if (longest * A.xcds > A.cap) return;  // the host allocates and runs this again
    int64_t b = blockIdx.x, first = 0, pos = 0;
    int piece = 0, len = -1;
    bool last = false;
    for (; piece < A.xcds; ++piece) {
        const int64_t k = A.start[piece + 1] - A.start[piece];
        const int64_t body = k > A.tail ? k - A.tail : 0;
        const int64_t nw = (body + A.window - 1) / A.window;
        if (b <= nw) {
            last = b == nw;
            pos = last ? body : b * A.window;
            first = A.start[piece] + pos;
            len = (int)(last ? k - body : (body - pos < A.window ? body - pos : A.window));
            break;
        }
        b -= nw + 1;
    }
    if (len < 0) return;
    int n2 = 1;
    while (n2 < len) n2 <<= 1;
    // padding sorts last: cost 0 and the largest group index
    uint64_t c = t < len ? A.cost[first + t] : 0;
    int32_t g = t < len ? (int32_t)(first + t) : 0x7fffffff;
    for (int size = 2; size <= n2; size <<= 1) {
        for (int stride = size >> 1; stride > 0; stride >>= 1) {
            uint64_t oc;
            int32_t og;
            if (stride >= 64) {
                __syncthreads();
                sc[t] = c;
                sg[t] = g;
                __syncthreads();
                oc = sc[t ^ stride];
                og = sg[t ^ stride];
            } else {
                oc = __shfl_xor((unsigned long long)c, stride);
                og = __shfl_xor(g, stride);
            }
            const bool want_first = ((t & stride) == 0) == ((t & size) == 0);
            if (costlier(c, g, oc, og) != want_first) {
                c = oc;
                g = og;
            }
        }
    }
    if (t < len) A.order[(pos + t) * A.xcds + piece] = g;
    if (last)
        for (int64_t k = pos + len + t; k < longest; k += kSortMax)
            A.order[k * A.xcds + piece] = -1;
}

}  // namespace

bool plan_order_device_supported(int window, int tail)
{
    return window >= 1 && window <= kSortMax && tail >= 0 && tail <= kSortMax;
}

// Scratch layout shared by the two calls below.
static PlanArgs plan_args(const ListPlan &P)
{
    PlanArgs A{};
    A.ng = P.ng;
    A.i_off = P.i_off;
    A.jp_cnt = P.jp_cnt;
    A.jc_cnt = P.jc_cnt;
    A.jp_off = P.jp_off;
    A.jc_off = P.jc_off;
    A.window = P.window;
    A.tail = P.tail;
    A.xcds = P.xcds;
    A.flag = P.flag;
    A.stats = P.stats;
    char *base = P.scratch->as<char>();
    A.start = reinterpret_cast<int64_t *>(base);
    A.cost = reinterpret_cast<uint64_t *>(base + (kMaxXcds + 1) * 8);
    A.tile = reinterpret_cast<Sums *>(base + (kMaxXcds + 1) * 8 + (size_t)P.ng * 8);
    A.order = P.order ? P.order->as<int32_t>() : nullptr;
    A.cap = P.order ? (int64_t)(P.order->cap / 4) : 0;
    return A;
}

static hipError_t launch_windows(const ListPlan &P, hipStream_t s)
{
    // windows: at most ng / window + 2 per piece
    const int64_t nwin = P.ng / P.window + 2 * (int64_t)P.xcds;
    hipLaunchKernelGGL(k_window_sort, dim3((unsigned)nwin), dim3(kSortMax), 0, s, plan_args(P));
    return hipGetLastError();
}

int plan_lists_launch(const ListPlan &P, hipStream_t s, std::string *what)
{
    auto fail = [&](hipError_t e) {
        *what = std::string("list plan: ") + hipGetErrorString(e);
        return e == hipErrorOutOfMemory ? BHQ_E_NOMEM : BHQ_E_HIP;
    };
    if (P.ng < 1 || P.xcds < 1 || P.xcds > kMaxXcds ||
        (P.order && !plan_order_device_supported(P.window, P.tail))) {
        *what = "list plan: bad argument";
        return BHQ_E_ARG;
    }
    const int64_t tiles = (P.ng + kTile - 1) / kTile;
    hipError_t e = P.scratch->reserve((kMaxXcds + 1) * 8 + (size_t)P.ng * 8 +
                                      (size_t)(tiles + 1) * sizeof(Sums));
    // pieces of equal cost are rarely longer than twice the mean
    if (e == hipSuccess && P.order)
        e = P.order->reserve(4 * (size_t)std::max<int64_t>(2 * P.ng, 64 * P.xcds));
    if (e != hipSuccess) return fail(e);
    const PlanArgs A = plan_args(P);
    if (tiles == 1) {
        hipLaunchKernelGGL(k_offsets<true>, dim3(2), dim3(kBlock), 0, s, A, 1);
    } else {
        hipLaunchKernelGGL(k_tile_sums, dim3((unsigned)tiles), dim3(kBlock), 0, s, A);
        if ((e = hipGetLastError()) != hipSuccess) return fail(e);
        hipLaunchKernelGGL(k_tile_scan, dim3(1), dim3(kBlock), 0, s, A, (int)tiles);
        if ((e = hipGetLastError()) != hipSuccess) return fail(e);
        hipLaunchKernelGGL(k_offsets<false>, dim3((unsigned)tiles), dim3(kBlock), 0, s, A,
                           (int)tiles);
    }
    e = hipGetLastError();
    if (e == hipSuccess && P.order) e = launch_windows(P, s);
    return e == hipSuccess ? BHQ_OK : fail(e);
}

int plan_lists_finish(const ListPlan &P, hipStream_t s, std::string *what)
{
    const int64_t slots = P.stats[kStatSlots];
    if (slots <= (int64_t)(P.order->cap / 4)) return BHQ_OK;
    hipError_t e = P.order->reserve((size_t)slots * 4);
    if (e == hipSuccess) e = launch_windows(P, s);
    if (e == hipSuccess) e = hipStreamSynchronize(s);
    if (e == hipSuccess) return BHQ_OK;
    *what = std::string("list plan: ") + hipGetErrorString(e);
    return e == hipErrorOutOfMemory ? BHQ_E_NOMEM : BHQ_E_HIP;
}

}  // namespace bhq
