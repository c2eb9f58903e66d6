// Stage 1: per-channel minimum / maximum / sum of a tall row-major matrix
// (Sec. 3.2: channel range and tensor range; Sec. 3.3: E[x] collected alongside).
//
// HBM-bound streaming pass (col_stats.hpp): each block leaves one partial row of (min, max, sum) in the workspace, and a second
// small kernel folds the slices in a fixed order (so the fp64 sums are reproducible) and merges with earlier batches.
#include "col_stats.hpp"
#include <atomic>

namespace aweq {

template <bool F16, bool KEEP>
__global__ __launch_bounds__(kStatsBlock) void col_stats_partial(
    const void* __restrict__ M, int64_t rows, int64_t K, int64_t ld, int64_t rows_per_slice,
    float* __restrict__ pmin, float* __restrict__ pmax, double* __restrict__ psum, uint32_t* __restrict__ ticket)
{
    __shared__ StatsLds<SliceStats<F16>::kCols> s;
    if (blockIdx.x == 0 && blockIdx.y == 0 && threadIdx.x == 0) *ticket = 0u;   // (for the merge kernel that follows on the stream)
    const int64_t r0 = (int64_t)blockIdx.y * rows_per_slice, o = (int64_t)blockIdx.y * K;
    stats_slice<F16>(s, M, K, ld, blockIdx.x, r0, min(rows, r0 + rows_per_slice), KEEP, pmin + o, pmax + o, psum + o);
}

// Fold the row slices and merge with what the caller already holds.  A block owns 32 columns;
// its 32 groups of 32 threads take every 32nd slice each (the kernel is bound by the latency of these
// few dependent loads, so they are spread over many threads) and meet in LDS in a fixed order, so
// the fp64 sums are reproducible.
// finalize: r = max - min per channel is written with the columns; R = tensor max - tensor min and
// p = r / R (Eq. 4) need every block's columns.  Each block leaves its extremes in its own (already read)
// columns of the first partial row, and a second small kernel finds R and writes p.  ONE: the last block, found by
// a ticket, does that in the same launch.  Every block's device-wide fence and atomic stands in a row with the others', so
// only few blocks do so (whole binary16 call, us, one launch / two: 64 tokens x 128 channels 10.2 / 11.4, 1 x 512 10.3 / 11.2,
// 1 x 1024 10.9 / 11.5; 4096 x 1280 14.2 / 11.4, 4096 x 2048 16.4 / 11.7).
constexpr int kMergeCols = 32, kMergeParts = 32;
constexpr int64_t kOneMergeK = 1024;
static_assert(kOneMergeK <= kMergeCols * kMergeCols && kOneMergeK <= kMergeCols * kMergeParts, "the last block reads an extreme a lane, a column a thread");
template <bool ONE>
__global__ __launch_bounds__(kMergeCols * kMergeParts) void col_stats_merge(
    float* pmin, float* pmax, const double* __restrict__ psum,
    int slices, int64_t K, int64_t rows, float* cmin, float* cmax,
    double* __restrict__ csum, uint64_t* __restrict__ count, int accumulate, uint32_t* status,
    int finalize, float* __restrict__ r, float* __restrict__ R, float* __restrict__ p, uint32_t* ticket)
{
    __shared__ int s_last;
    __shared__ float s_a[kMergeParts][kMergeCols], s_b[kMergeParts][kMergeCols];
    __shared__ double s_s[kMergeParts][kMergeCols];
    const int c = threadIdx.x & (kMergeCols - 1), part = threadIdx.x / kMergeCols;
    const int64_t k = (int64_t)blockIdx.x * kMergeCols + c;
    if (blockIdx.x == 0 && threadIdx.x == 0 && count) *count = (accumulate ? *count : 0ull) + (uint64_t)rows;
    float a = INFINITY, b = -INFINITY;
    double s = 0.0;
    if (k < K)
        for (int j = part; j < slices; j += kMergeParts) {
            a = fminf(a, pmin[(int64_t)j * K + k]);
            b = fmaxf(b, pmax[(int64_t)j * K + k]);
            s += psum[(int64_t)j * K + k];
        }
    s_a[part][c] = a; s_b[part][c] = b; s_s[part][c] = s;
    __syncthreads();
    if (part == 0 && k < K) {
#pragma unroll
        for (int q = 1; q < kMergeParts; ++q) {
            a = fminf(a, s_a[q][c]);
            b = fmaxf(b, s_b[q][c]);
            s += s_s[q][c];
        }
        // a non-finite input makes the fp64 sum (Inf / NaN) or an extreme (Inf) non-finite
        if (!isfinite(s) || isinf(a) || isinf(b)) raise_status(status, AWEQ_ST_NONFINITE);
        if (accumulate) {
            a = fminf(a, cmin[k]);
            b = fmaxf(b, cmax[k]);
            if (csum) s += csum[k];
        }
        cmin[k] = a;
        cmax[k] = b;
        if (csum) csum[k] = s;
        if (finalize) r[k] = b - a;
    }
    if (finalize && part == 0) {
        // this block's extremes (lanes past K hold the identities)
        a = group_allreduce<5>(k < K ? a : INFINITY, OpMin());
        b = group_allreduce<5>(k < K ? b : -INFINITY, OpMax());
        if (c == 0) {
            pmin[k] = a;
            pmax[k] = b;
            if constexpr (ONE) {
                __threadfence();   // the extremes and this wavefront's r are visible device-wide before the ticket is
                s_last = atomicAdd(ticket, 1u) == gridDim.x - 1;
            }
        }
    }
    if constexpr (ONE) {
        if (!finalize) return;
        __syncthreads();
        if (!s_last) return;
        __threadfence();           // every other block's extremes and r are visible to this one
        auto seen = [](const float* q) { return __hip_atomic_load(q, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); };
        const bool ratio = p && (int64_t)threadIdx.x < K;
        const float rk = ratio ? seen(&r[threadIdx.x]) : 0.0f;
        const bool some = c < (int)gridDim.x;
        a = group_allreduce<5>(some ? seen(&pmin[c * kMergeCols]) : INFINITY, OpMin());
        b = group_allreduce<5>(some ? seen(&pmax[c * kMergeCols]) : -INFINITY, OpMax());
        const float RR = (b - a) + 0.0f;
        if (threadIdx.x == 0) *R = RR;
        if (ratio) p[threadIdx.x] = rk / RR;
    }
}

// R and p from the extremes the merge kernel's blocks left at every kMergeCols-th column
constexpr int kFinishBlock = 256;
__global__ __launch_bounds__(kFinishBlock) void col_stats_finish(
    const float* __restrict__ bmin, const float* __restrict__ bmax, int64_t K, const float* __restrict__ r,
    float* __restrict__ R, float* __restrict__ p)
{
    __shared__ float slot[kFinishBlock / kWave];
    const int64_t k = (int64_t)blockIdx.x * kFinishBlock + threadIdx.x;
    const float rk = k < K ? r[k] : 0.0f;
    float a = INFINITY, b = -INFINITY;
    for (int64_t j = (int64_t)threadIdx.x * kMergeCols; j < K; j += (int64_t)kFinishBlock * kMergeCols) {
        a = fminf(a, bmin[j]);
        b = fmaxf(b, bmax[j]);
    }
    a = block_allreduce<kFinishBlock / kWave>(a, OpMin(), slot);
    b = block_allreduce<kFinishBlock / kWave>(b, OpMax(), slot);
    const float RR = (b - a) + 0.0f;   // (a tensor of zeros of both signs has range +0)
    if (k == 0) *R = RR;
    if (p && k < K) p[k] = rk / RR;
}

size_t stats_ws_bytes_export(int64_t rows, int64_t K) { return stats_ws_bytes(rows, K); }

// the statistics pass on a workspace that is known to be large enough and 16-byte aligned
static int run_calib_stats(const void* M, aweq_dtype dt, int64_t rows, int64_t K, int64_t ld,
                           float* cmin, float* cmax, double* csum, uint64_t* count,
                           int accumulate, int finalize, float* r, float* R, float* p,
                           void* ws, uint32_t* status, hipStream_t st)
{
    const int epl = dt == AWEQ_F16 ? 8 : 4;
    const StatsPlan plan = stats_plan(rows, K, epl);
    // workspace layout: psum (fp64) first, then pmin, pmax
    double* psum = reinterpret_cast<double*>(ws);
    float* pmin = reinterpret_cast<float*>(psum + (size_t)plan.slices * K);
    float* pmax = pmin + (size_t)plan.slices * K;
    uint32_t* ticket = reinterpret_cast<uint32_t*>(pmax + (size_t)plan.slices * K);
    dim3 grid(plan.col_chunks, plan.slices);
    // A matrix that fits the memory-side cache together with what the next pass over it writes (the folded weight and its codes: 2.5
    // times its size) is read through the caches, where that pass finds it: fold + quantise 4096 x 11008 (90 MB) 51.0 -> 42.9 us,
    // the fold alone 29.9 -> 27.7, this pass 17.2 -> 16.0 there; seven sequences through the calibration 249.9 -> 239.8.  On matrices in
    // neither cache the two kinds of loads take the same up to 90 MB (25.9 / 26.1 us with the merge), beyond it plain ones
    // are slower (134 MB 35.0 -> 36.1, 262 MB 53.1 -> 55.7).
    const bool keep = rows * K * (int64_t)dtype_size(dt) <= kKeepBytes;
#define AWEQ_CS(F, P) col_stats_partial<F, P><<<grid, kStatsBlock, 0, st>>>(M, rows, K, ld, plan.rows_per_slice, pmin, pmax, psum, ticket)
    if (dt == AWEQ_F16) { if (keep) AWEQ_CS(true, true); else AWEQ_CS(true, false); }
    else { if (keep) AWEQ_CS(false, true); else AWEQ_CS(false, false); }
#undef AWEQ_CS
    const bool one = finalize && K <= kOneMergeK;
    const unsigned blocks = (unsigned)cdiv(K, kMergeCols);
#define AWEQ_CM(ONE) col_stats_merge<ONE><<<blocks, kMergeCols * kMergeParts, 0, st>>>(pmin, pmax, psum, plan.slices, K, rows, cmin, cmax, csum, count, accumulate, status, finalize, r, R, p, ticket)
    if (one) AWEQ_CM(true); else AWEQ_CM(false);
#undef AWEQ_CM
    if (finalize && !one) col_stats_finish<<<(unsigned)cdiv(p ? K : 1, kFinishBlock), kFinishBlock, 0, st>>>(pmin, pmax, K, r, R, p);
    return launch_status();
}

static int check_calib_stats_args(const void* M, aweq_dtype dt, int64_t rows, int64_t K, int64_t ld,
                                  const float* cmin, const float* cmax, int finalize, const float* r, const float* R)
{
    if (!M || !cmin || !cmax) return AWEQ_ERR_NULL;
    if (finalize && (!r || !R)) return AWEQ_ERR_NULL;
    if (dt != AWEQ_F32 && dt != AWEQ_F16) return AWEQ_ERR_DTYPE;
    if (rows <= 0 || K <= 0 || ld < K || (K % 8) != 0) return AWEQ_ERR_SHAPE;
    if (!aligned16(M) || ((size_t)ld * dtype_size(dt)) % 16 != 0) return AWEQ_ERR_ALIGN;
    return AWEQ_OK;
}

// ---- scratch of the entry point that may not allocate: the per-slice partial rows live in a
// file-scope device array instead of a caller's workspace.  Every GPU the library runs on holds
// its own copy of the array (at its own address) until the process ends.
constexpr size_t kStaticScratchBytes = AWEQ_STATIC_SCRATCH_BYTES;
static __device__ __align__(256) unsigned char scratch[kStaticScratchBytes];

constexpr int kMaxDevices = 64;
static std::atomic<void*> g_scratch_of_device[kMaxDevices];

// device address of `scratch` on the current device (looked up once per device; in host code the
// array's name is only a handle for this lookup, never an address a kernel may be given)
static int static_scratch(void** out)
{
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return AWEQ_ERR_LAUNCH;
    void* ptr = g_scratch_of_device[dev].load(std::memory_order_acquire);
    if (!ptr) {
        if (hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)) != hipSuccess || !ptr) return AWEQ_ERR_LAUNCH;
        g_scratch_of_device[dev].store(ptr, std::memory_order_release);   // (a racing thread stores the same address)
    }
    *out = ptr;
    return AWEQ_OK;
}

}  // namespace aweq

using namespace aweq;

extern "C" int aweq_calib_stats(const void* M, aweq_dtype dt, int64_t rows, int64_t K, int64_t ld,
                                float* cmin, float* cmax, double* csum, uint64_t* count,
                                int accumulate, int finalize, float* r, float* R, float* p,
                                void* ws, size_t ws_bytes, uint32_t* status, void* stream)
{
    const int rc = check_calib_stats_args(M, dt, rows, K, ld, cmin, cmax, finalize, r, R);
    if (rc != AWEQ_OK) return rc;
    if (!ws || ws_bytes < stats_ws_bytes(rows, K)) return AWEQ_ERR_WORKSPACE;
    if (!aligned16(ws)) return AWEQ_ERR_ALIGN;
    return run_calib_stats(M, dt, rows, K, ld, cmin, cmax, csum, count, accumulate, finalize, r, R, p, ws, status,
                           as_stream(stream));
}

extern "C" int aweq_calib_stats_static(const void* M, aweq_dtype dt, int64_t rows, int64_t K, int64_t ld,
                                       float* cmin, float* cmax, double* csum, uint64_t* count,
                                       int accumulate, int finalize, float* r, float* R, float* p,
                                       uint32_t* status, void* stream)
{
    const int rc = check_calib_stats_args(M, dt, rows, K, ld, cmin, cmax, finalize, r, R);
    if (rc != AWEQ_OK) return rc;
    if (stats_ws_bytes(rows, K) > kStaticScratchBytes) return AWEQ_ERR_WORKSPACE;   // beyond the built-in scratch
    void* ptr = nullptr;
    const int src = static_scratch(&ptr);
    if (src != AWEQ_OK) return src;
    // every partial row the merge reads and its ticket are written by this call's first
    // kernel: the array's contents from earlier calls never matter and nothing has to be cleared
    return run_calib_stats(M, dt, rows, K, ld, cmin, cmax, csum, count, accumulate, finalize, r, R, p, ptr, status,
                           as_stream(stream));
}
