// bhq_sort.h -- stable sort of up to kRankSortMost (key, index) pairs by key
// bits (device code), for the sizes at which a device sort's time is its
// launches: blocks sort tiles of 1024 to 4096 keys, which they read or form
// themselves, and one or two launches merge up to eight sorted runs each,
// every element finding its place by its rank in the other runs.
//
// Bound by the chain of dependent loads of the ranks' binary searches; the
// up to eight searches of an element go side by side (one after another they
// took three times as long).  Keys of 18 bits, 64 / 32 wide, with the keys
// formed before, against the library's sort, whose merge levels are a launch
// or two each (us): 2,000 10 / 10 and 15 / 14, 16,384 20 / 17 and 26 / 25,
// 65,536 28 / 23 and 41 / 38, 131,072 35 / 29 and 57 / 51, 216,000 55 / 44 and
// 98 / 90; of 63 bits, 131,072 48 and 66, 216,000 79 and 106.  The tile grows
// with n so that two merges do up to 2^18 (three merges of smaller tiles, or
// larger tiles where they are not needed, were slower); beyond, the library's
// sort by digits is as fast.
#pragma once

#include <hip/hip_runtime.h>
#include <hipcub/hipcub.hpp>

#include <cstdint>

namespace bhq {

constexpr int64_t kRankSortMost = 262144;
constexpr int kRankWays = 8;

// Keys formed before (they may be in the array that rank_sort takes as
// scratch: a tile is read before it is written).
template <typename K>
struct StoredKeys {
    const K *key;
    __device__ __forceinline__ K operator()(int p) const { return key[p]; }
};

// Sorted tiles of (make(p), p) on key bits [b0, b1).
template <typename K, int BS, int IT, typename Make>
__global__ __launch_bounds__(BS) void k_tile_sort(const Make make, int n, int b0, int b1, K *ko,
                                                  int32_t *vo)
{
    typedef hipcub::BlockRadixSort<K, BS, IT, int32_t> Sort;
    __shared__ typename Sort::TempStorage tmp;
    const int base = (int)blockIdx.x * BS * IT, t = threadIdx.x;
    K k[IT];
    int32_t v[IT];
#pragma unroll
    for (int u = 0; u < IT; ++u) {
        // what is past the end stays behind its equals (the sort is stable)
        const int p = base + t * IT + u;
        k[u] = p < n ? make(p) : (K)~(K)0;
        v[u] = p;
    }
    Sort(tmp).SortBlockedToStriped(k, v, b0, b1);
#pragma unroll
    for (int u = 0; u < IT; ++u) {
        const int p = base + u * BS + t;
        if (p < n) {
            ko[p] = k[u];
            vo[p] = v[u];
        }
    }
}

// Sorted runs of `len` (the last one shorter), `ways` <= kRankWays of them to
// one.  Keys are compared from bit lo up and are less than all ones there.
template <typename K>
__global__ __launch_bounds__(256) void k_rank_merge(const K *k, const int32_t *v, int n, int lo,
                                                    int len, int ways, K *ko, int32_t *vo)
{
    const int i = (int)(blockIdx.x * 256 + threadIdx.x);
    if (i >= n) return;
    const K key = k[i], c = key >> lo;
    const int run = i / len, r0 = run / ways * ways, own = run - r0;
    // per run: entries, entries known to come before this one, the limit (one
    // more in the runs before, whose equals come first), and the address
    // before the first entry (of the element itself where there is none, so
    // that every load is in bounds and none waits for another's test)
    int cnt[kRankWays], at[kRankWays], base[kRankWays];
    K lim[kRankWays];
#pragma unroll
    for (int q = 0; q < kRankWays; ++q) {
        const int64_t a = (int64_t)(r0 + q) * len;
        const bool use = q < ways && q != own && a < n;
        cnt[q] = use ? (int)(n - a < len ? n - a : len) : 0;
        base[q] = use ? (int)a - 1 : i - 1;
        lim[q] = c + (q < own ? 1 : 0);
        at[q] = 0;
    }
    int step = 1;
    while (step < len) step *= 2;
    for (; step > 0; step /= 2) {
        K x[kRankWays];
#pragma unroll
        for (int q = 0; q < kRankWays; ++q) {
            const int p = at[q] + step, last = cnt[q] > 1 ? cnt[q] : 1;
            x[q] = k[base[q] + (p < last ? p : last)] >> lo;
        }
#pragma unroll
        for (int q = 0; q < kRankWays; ++q) {
            const int p = at[q] + step;
            if (p <= cnt[q] && x[q] < lim[q]) at[q] = p;
        }
    }
    int pos = i - own * len;
#pragma unroll
    for (int q = 0; q < kRankWays; ++q) pos += at[q];
    ko[pos] = key;
    vo[pos] = v[i];
}

// Stable sort of the pairs (make(p), p), 0 <= p < n <= kRankSortMost, on key
// bits [b0, b1) to k1, v1; k0, v0 are scratch.  make gives keys without bits
// from b1 up, b1 less than the width of K.
template <typename K, typename Make>
hipError_t rank_sort(const Make &make, int64_t n, int b0, int b1, K *k0, int32_t *v0, K *k1,
                     int32_t *v1, hipStream_t s)
{
    if (n > kRankSortMost || b1 >= (int)(8 * sizeof(K))) return hipErrorInvalidValue;
    const int m = (int)n;
    // tile, so that one merge (up to 8 tiles of 2048) or two (64 tiles) do
    const int tile = m <= 16384 ? 2048 : m <= 65536 ? 1024 : m <= 131072 ? 2048 : 4096;
    const int runs = (m + tile - 1) / tile;
    const int merges = runs <= 1 ? 0 : runs <= kRankWays ? 1 : 2;
    int ways = merges == 1 ? runs : 1;
    if (merges == 2)
        while (ways * ways < runs) ++ways;
    K *ka = merges == 1 ? k0 : k1, *kb = merges == 1 ? k1 : k0;
    int32_t *va = merges == 1 ? v0 : v1, *vb = merges == 1 ? v1 : v0;
    const dim3 g((unsigned)runs), gm((unsigned)((m + 255) / 256));
    if (tile == 1024)
        hipLaunchKernelGGL((k_tile_sort<K, 256, 4, Make>), g, dim3(256), 0, s, make, m, b0, b1, ka,
                           va);
    else if (tile == 2048)
        hipLaunchKernelGGL((k_tile_sort<K, 512, 4, Make>), g, dim3(512), 0, s, make, m, b0, b1, ka,
                           va);
    else
        hipLaunchKernelGGL((k_tile_sort<K, 1024, 4, Make>), g, dim3(1024), 0, s, make, m, b0, b1,
                           ka, va);
    int len = tile;
    for (int i = 0; i < merges; ++i) {
        hipLaunchKernelGGL(k_rank_merge<K>, gm, dim3(256), 0, s, ka, va, m, b0, len, ways, kb, vb);
        len *= ways;
        K *kt = ka;
        ka = kb, kb = kt;
        int32_t *vt = va;
        va = vb, vb = vt;
    }
    return hipGetLastError();
}

}  // namespace bhq
