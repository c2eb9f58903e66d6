// Column minimum / maximum / sum over one row slice of a row-major matrix: the streaming pass that the statistics entry point and the
// calibration of a whole layer share.  Lanes own columns (16 bytes = 8 halves or 4 floats per lane), so a wavefront reads 1 KiB
// contiguous per row; the four wavefronts of a block take interleaved rows of a slice and meet in LDS; each block writes one partial
// row of (min, max, sum).
#pragma once
#include "common.hpp"

namespace aweq {

constexpr int kStatsBlock = 256;
constexpr int kStatsWaves = kStatsBlock / kWave;
constexpr int kRowBatch = 8;  // rows summed in fp32 before one fp64 add (binary16 input only)

// Heights of slices that blocks walk down side by side: no multiple of 64 rows.  With rows of a power of two of bytes the slices would begin a
// multiple of a large power of two apart and the blocks would be at the same memory channels all along (us, whole calibration, 512 -> 544 rows a
// slice: 32768 x 4096 144 -> 127, 61440 x 4096 209 -> 197, 28672 x 16384 423 -> 412).
inline int64_t spread_rows(int64_t rows) { return rows >= 64 && rows % 64 == 0 ? rows + 32 : rows; }

struct StatsPlan {
    int col_chunks;   // blocks along K
    int slices;       // row slices
    int64_t rows_per_slice;
};

// Same plan on the host for the launch and for the workspace size.
inline StatsPlan stats_plan(int64_t rows, int64_t K, int elts_per_lane)
{
    StatsPlan p;
    const int64_t cols_per_block = (int64_t)kWave * elts_per_lane;
    p.col_chunks = (int)cdiv(K, cols_per_block);
    int64_t want = cdiv(1280, p.col_chunks);           // 5 blocks per compute unit, all resident: fewer partial rows to merge
    int64_t max_slices = cdiv(rows, kStatsWaves * kRowBatch);  // at least one row batch per wavefront
    if (want > max_slices) want = max_slices;
    if (want < 1) want = 1;
    p.rows_per_slice = spread_rows(cdiv(cdiv(rows, want), kStatsWaves * kRowBatch) * (kStatsWaves * kRowBatch));
    p.slices = (int)cdiv(rows, p.rows_per_slice);
    return p;
}

inline size_t stats_ws_bytes(int64_t rows, int64_t K)
{
    // sized for the narrower lane width (more chunks never increases the slice count)
    StatsPlan a = stats_plan(rows, K, 8), b = stats_plan(rows, K, 4);
    int s = a.slices > b.slices ? a.slices : b.slices;
    return (size_t)s * (size_t)K * (sizeof(float) * 2 + sizeof(double)) + 16;   // partial rows, then the merge kernel's ticket
}

constexpr int64_t kKeepBytes = kCacheBytes * 3 / 8;

// Every byte of the matrix is read exactly once by this pass.  KEEP: through the caches, for the pass that reads the same matrix next
// (rule and figures at the launch); otherwise non-temporal.
template <bool KEEP>
__device__ __forceinline__ Half8 load_once(const _Float16* p)
{
    typedef int v4i_ __attribute__((ext_vector_type(4)));
    const v4i_* const q = reinterpret_cast<const v4i_*>(p);
    return __builtin_bit_cast(Half8, KEEP ? *q : __builtin_nontemporal_load(q));
}
template <bool KEEP>
__device__ __forceinline__ Float4 load_once(const float* p)
{
    typedef float v4f_ __attribute__((ext_vector_type(4)));
    const v4f_* const q = reinterpret_cast<const v4f_*>(p);
    return __builtin_bit_cast(Float4, KEEP ? *q : __builtin_nontemporal_load(q));
}

// extremes and sums of a block's wavefronts.  (16 bytes: aligned to their doubles only they were written 8 bytes at a time, binary16
// 1000 x 11008 13.4 -> 12.7 us)
template <int E>
struct alignas(16) StatsLds {
    float mn[kStatsWaves][kWave][E], mx[kStatsWaves][kWave][E];
    double sm[kStatsWaves][kWave][E];
};

template <bool F16> struct SliceStats;

// ---- binary16: 8 columns per lane, kRowBatch rows added in binary32 before one fp64 add
template <>
struct SliceStats<true> {
    static constexpr int kCols = 8;
    f16x2 mn[4], mx[4];
    double sum[8];
    __device__ __forceinline__ SliceStats()
    {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            mn[i] = f16x2{(_Float16)INFINITY, (_Float16)INFINITY};
            mx[i] = f16x2{(_Float16)-INFINITY, (_Float16)-INFINITY};
        }
#pragma unroll
        for (int i = 0; i < 8; ++i) sum[i] = 0.0;
    }
    __device__ __forceinline__ void put(int i, float& a, float& b) const   // column i's extremes
    {
        a = (float)(i & 1 ? mn[i >> 1].y : mn[i >> 1].x);
        b = (float)(i & 1 ? mx[i >> 1].y : mx[i >> 1].x);
    }
    // wavefront w takes rows r_begin + w, + kStatsWaves, ...; kRowBatch rows in flight
    template <bool KEEP>
    __device__ __forceinline__ void add_rows(const void* Mv, int64_t ld, int64_t col, int64_t r, int64_t r_end)
    {
        const _Float16* const base = reinterpret_cast<const _Float16*>(Mv) + col;
        for (; r + (int64_t)(kRowBatch - 1) * kStatsWaves < r_end; r += (int64_t)kRowBatch * kStatsWaves) {
            Half8 v[kRowBatch];
#pragma unroll
            for (int j = 0; j < kRowBatch; ++j)
                v[j] = load_once<KEEP>(base + (r + (int64_t)j * kStatsWaves) * ld);
            float part[8] = {0, 0, 0, 0, 0, 0, 0, 0};
#pragma unroll
            for (int j = 0; j < kRowBatch; ++j)
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    mn[i] = hmin2(mn[i], v[j].h[i]);
                    mx[i] = hmax2(mx[i], v[j].h[i]);
                    float2 f = h2f2(v[j].h[i]);
                    part[2 * i] += f.x;
                    part[2 * i + 1] += f.y;
                }
#pragma unroll
            for (int i = 0; i < 8; ++i) sum[i] += (double)part[i];
        }
        for (; r < r_end; r += kStatsWaves) {
            Half8 v = load_once<KEEP>(base + r * ld);
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                mn[i] = hmin2(mn[i], v.h[i]);
                mx[i] = hmax2(mx[i], v.h[i]);
                float2 f = h2f2(v.h[i]);
                sum[2 * i] += (double)f.x;
                sum[2 * i + 1] += (double)f.y;
            }
        }
    }
};

// ---- binary32: 4 columns per lane, every element added in fp64
template <>
struct SliceStats<false> {
    static constexpr int kCols = 4;
    float mn[4], mx[4];
    double sum[4];
    __device__ __forceinline__ SliceStats()
    {
#pragma unroll
        for (int i = 0; i < 4; ++i) { mn[i] = INFINITY; mx[i] = -INFINITY; sum[i] = 0.0; }
    }
    __device__ __forceinline__ void put(int i, float& a, float& b) const { a = mn[i]; b = mx[i]; }
    template <bool KEEP>
    __device__ __forceinline__ void add_rows(const void* Mv, int64_t ld, int64_t col, int64_t r, int64_t r_end)
    {
        const float* const base = reinterpret_cast<const float*>(Mv) + col;
        for (; r + (int64_t)(kRowBatch - 1) * kStatsWaves < r_end; r += (int64_t)kRowBatch * kStatsWaves) {
            Float4 v[kRowBatch];
#pragma unroll
            for (int j = 0; j < kRowBatch; ++j)
                v[j] = load_once<KEEP>(base + (r + (int64_t)j * kStatsWaves) * ld);
#pragma unroll
            for (int j = 0; j < kRowBatch; ++j)
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    mn[i] = fminf(mn[i], v[j].f[i]);
                    mx[i] = fmaxf(mx[i], v[j].f[i]);
                    sum[i] += (double)v[j].f[i];
                }
        }
        for (; r < r_end; r += kStatsWaves) {
            Float4 v = load_once<KEEP>(base + r * ld);
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                mn[i] = fminf(mn[i], v.f[i]);
                mx[i] = fmaxf(mx[i], v.f[i]);
                sum[i] += (double)v.f[i];
            }
        }
    }
};

// The partial row of rows [r_begin, r_end) in column chunk `chunk` (kWave lanes of columns), written to prow_*[K].
// One block of kStatsBlock threads.
template <bool F16>
__device__ __forceinline__ void stats_slice(StatsLds<SliceStats<F16>::kCols>& s, const void* M, int64_t K, int64_t ld, int chunk,
                                            int64_t r_begin, int64_t r_end, bool keep, float* __restrict__ prow_min,
                                            float* __restrict__ prow_max, double* __restrict__ prow_sum)
{
    constexpr int E = SliceStats<F16>::kCols;
    const int lane = threadIdx.x & (kWave - 1);
    const int wave = threadIdx.x / kWave;
    const int64_t col = ((int64_t)chunk * kWave + lane) * E;
    SliceStats<F16> p;
    if (col < K) {
        if (keep) p.template add_rows<true>(M, ld, col, r_begin + wave, r_end);
        else p.template add_rows<false>(M, ld, col, r_begin + wave, r_end);
    }
#pragma unroll
    for (int i = 0; i < E; ++i) {
        p.put(i, s.mn[wave][lane][i], s.mx[wave][lane][i]);
        s.sm[wave][lane][i] = p.sum[i];
    }
    __syncthreads();
    for (int c = threadIdx.x; c < kWave * E; c += kStatsBlock) {
        const int l = c / E, i = c % E;
        float a = s.mn[0][l][i], b = s.mx[0][l][i];
        double sm = s.sm[0][l][i];
#pragma unroll
        for (int w = 1; w < kStatsWaves; ++w) {
            a = fminf(a, s.mn[w][l][i]);
            b = fmaxf(b, s.mx[w][l][i]);
            sm += s.sm[w][l][i];
        }
        const int64_t k = (int64_t)chunk * kWave * E + c;
        if (k < K) { prow_min[k] = a; prow_max[k] = b; prow_sum[k] = sm; }
    }
}

}  // namespace aweq
