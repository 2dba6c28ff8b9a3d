// bhq_upload.hip -- device-side uploads for the set calls that read caller
// device memory (bhq_set_*_dev): validation of the caller's arrays into a
// flag word, and their copy into the context's layout (AoS columns to SoA
// arrays, pool records).  Every kernel only reads its inputs and writes the
// context's arrays; nothing is decided here that the host calls decide
// differently.
//
// A set call is latency: its arrays are checked in one launch and copied in
// another, which does nothing if the checks failed, so the host waits once.
// With a launch per array, library copies and a wait between the checks and
// the copies, setting 301 groups and their lists took about 300 us.
#include <hip/hip_runtime.h>

#include <cmath>

#include "bhq_internal.h"

namespace bhq {

namespace {

constexpr int kBlock = 256;

inline unsigned grid(int64_t n)
{
    const int64_t b = (n + kBlock - 1) / kBlock;
    return (unsigned)(b < 65535 * 16 ? (b > 0 ? b : 1) : 65535 * 16);
}

__global__ __launch_bounds__(kBlock) void k_clear(unsigned *flag)
{
    if (blockIdx.x == 0 && threadIdx.x == 0) *flag = 0u;
}

struct Columns {
    UploadCol c[kMaxUploadCols];
    int n;
};

// All of a call's arrays in one pass, a row of blocks for each.
__global__ __launch_bounds__(kBlock) void k_check_cols(const Columns C, unsigned *flag)
{
    const UploadCol &u = C.c[blockIdx.y];
    if (!u.src) return;
    unsigned bad = 0;
    const int64_t total = u.n * u.w, step = (int64_t)gridDim.x * kBlock;
    for (int64_t k = (int64_t)blockIdx.x * kBlock + threadIdx.x; k < total; k += step) {
        if (u.kind == kColOffsets) {
            // off[0] == 0 and off[g] <= off[g + 1]
            const int64_t *off = static_cast<const int64_t *>(u.src);
            if (k == 0 ? off[0] != 0 : off[k] < off[k - 1]) bad |= kBadOrder;
        } else {
            const double x = static_cast<const double *>(u.src)[k];
            if (!isfinite(x)) bad |= kBadNonFinite;
            else if (u.kind == kColPositive && !(x >= kMinEps2)) bad |= kBadNonPositive;
        }
    }
    if (bad) atomicOr(flag, bad);
}

// Elements in memory order: coalesced reads, columns written in parts.
template <int W>
__device__ __forceinline__ void copy_cols(const UploadCol &u)
{
    const int64_t total = u.n * W, step = (int64_t)gridDim.x * kBlock;
    for (int64_t k = (int64_t)blockIdx.x * kBlock + threadIdx.x; k < total; k += step) {
        const int64_t row = k / W;
        const int col = (int)(k - row * W);
        const uint64_t v = u.src ? static_cast<const uint64_t *>(u.src)[k] : 0;
        if (u.dst[col]) static_cast<uint64_t *>(u.dst[col])[row] = v;
    }
}

// The arrays' columns to their places, unless a check failed (src NULL:
// zeros).  Publishes the flag to the host and clears the next call's.
__global__ __launch_bounds__(kBlock) void k_copy_cols(const Columns C, const unsigned *flag,
                                                      unsigned *next, unsigned *host)
{
    const unsigned bad = *flag;
    if (blockIdx.x == 0 && blockIdx.y == 0 && threadIdx.x == 0) {
        *host = bad;
        *next = 0u;
    }
    if (bad) return;
    const UploadCol &u = C.c[blockIdx.y];
    if (u.w == 1)
        copy_cols<1>(u);
    else if (u.w == 3)
        copy_cols<3>(u);
    else
        copy_cols<6>(u);
}

// Publishes the flag and the last offsets of a set of groups (three arrays).
__global__ void k_publish_groups(const Columns C, const unsigned *flag, unsigned *next,
                                 unsigned *host, int64_t *last)
{
    if (threadIdx.x == 0) {
        *host = *flag;
        *next = 0u;
    }
    if (threadIdx.x < 3) {
        const UploadCol &u = C.c[threadIdx.x];
        last[threadIdx.x] = static_cast<const int64_t *>(u.src)[u.n - 1];
    }
}

__global__ __launch_bounds__(kBlock) void k_check_idx(const int32_t *idx, int64_t n, int64_t pool,
                                                      unsigned *flag)
{
    unsigned bad = 0;
    for (int64_t k = (int64_t)blockIdx.x * kBlock + threadIdx.x; k < n;
         k += (int64_t)gridDim.x * kBlock) {
        const int32_t v = idx[k];
        if (v < 0 || (int64_t)v >= pool) bad |= kBadRange;
    }
    if (bad) atomicOr(flag, bad);
}

__global__ __launch_bounds__(kBlock) void k_pack_particles(const double *x, const double *m,
                                                           int64_t n, PartRec *out)
{
    for (int64_t k = (int64_t)blockIdx.x * kBlock + threadIdx.x; k < n;
         k += (int64_t)gridDim.x * kBlock)
        out[k] = PartRec{x[3 * k], x[3 * k + 1], x[3 * k + 2], m[k]};
}

__global__ __launch_bounds__(kBlock) void k_pack_cells(const double *x, const double *m,
                                                       const double *q, const double *t,
                                                       int64_t n, CellRec *out)
{
    for (int64_t k = (int64_t)blockIdx.x * kBlock + threadIdx.x; k < n;
         k += (int64_t)gridDim.x * kBlock) {
        const double *qk = q + 6 * k;
        out[k] = CellRec{x[3 * k], x[3 * k + 1], x[3 * k + 2], m[k], qk[0], qk[1], qk[2],
                         qk[3], qk[4], qk[5], t ? t[k] : 0.0, 0.0};
    }
}

}  // namespace

hipError_t launch_clear_flag(unsigned *flag, hipStream_t s)
{
    hipLaunchKernelGGL(k_clear, dim3(1), dim3(kBlock), 0, s, flag);
    return hipGetLastError();
}

static Columns columns(const UploadCol *c, int n, dim3 &g)
{
    Columns C{};
    C.n = n;
    int64_t most = 1;
    for (int k = 0; k < n; ++k) {
        C.c[k] = c[k];
        if (c[k].n * c[k].w > most) most = c[k].n * c[k].w;
    }
    // four elements a thread: the blocks of short columns end at once
    g = dim3(grid((most + 3) / 4), (unsigned)n);
    return C;
}

hipError_t launch_check_cols(const UploadCol *c, int n, unsigned *flag, hipStream_t s)
{
    if (n < 1 || n > kMaxUploadCols) return hipErrorInvalidValue;
    dim3 g;
    const Columns C = columns(c, n, g);
    hipLaunchKernelGGL(k_check_cols, g, dim3(kBlock), 0, s, C, flag);
    return hipGetLastError();
}

hipError_t launch_copy_cols(const UploadCol *c, int n, const unsigned *flag, unsigned *next,
                            unsigned *host, hipStream_t s)
{
    if (n < 1 || n > kMaxUploadCols) return hipErrorInvalidValue;
    for (int k = 0; k < n; ++k)
        if (c[k].w != 1 && c[k].w != 3 && c[k].w != 6) return hipErrorInvalidValue;
    dim3 g;
    const Columns C = columns(c, n, g);
    hipLaunchKernelGGL(k_copy_cols, g, dim3(kBlock), 0, s, C, flag, next, host);
    return hipGetLastError();
}

hipError_t launch_publish_groups(const UploadCol *c, const unsigned *flag, unsigned *next,
                                 unsigned *host, int64_t *last, hipStream_t s)
{
    dim3 g;
    hipLaunchKernelGGL(k_publish_groups, dim3(1), dim3(64), 0, s, columns(c, 3, g), flag, next,
                       host, last);
    return hipGetLastError();
}

hipError_t launch_check_idx(const int32_t *idx, int64_t n, int64_t pool, unsigned *flag,
                            hipStream_t s)
{
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_check_idx, dim3(grid(n)), dim3(kBlock), 0, s, idx, n, pool, flag);
    return hipGetLastError();
}

hipError_t launch_pack_particles(const double *x, const double *m, int64_t n, PartRec *out,
                                 hipStream_t s)
{
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_pack_particles, dim3(grid(n)), dim3(kBlock), 0, s, x, m, n, out);
    return hipGetLastError();
}

hipError_t launch_pack_cells(const double *x, const double *m, const double *q,
                             const double *t, int64_t n, CellRec *out, hipStream_t s)
{
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_pack_cells, dim3(grid(n)), dim3(kBlock), 0, s, x, m, q, t, n, out);
    return hipGetLastError();
}

}  // namespace bhq
