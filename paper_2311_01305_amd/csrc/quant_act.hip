// Stage 4a: static per-tensor int8 activation quantizer (Sec. 2, Eq. 1 with b = 8) applied
// to the equalised activation X_hat = X diag(s)^-1 (Sec. 3.1, Eq. 3) on the fly, with the
// per-token and per-channel code sums the GEMM epilogue and the bias correction need.
//
// HBM-bound (2 bytes in, 1 byte out per element for binary16) with a tight ALU budget, so
// the quotient x / Step is formed without the generic division sequence when that is
// provably the same: Step is one constant, y = RN(1 / Step) is computed once, and
//   q0 = RN(a y);  r = a - Step q (exact, FMA);  q = RN(q + r y)   applied twice
// gives the correctly rounded a / Step.  After the first correction q is within
// 1/2 + 2^-22 ulp of a / Step; a quotient of two binary32 numbers is at least
// 2^-25 / beta ulp away from a rounding boundary (beta = significand(Step) / 2^24 < 1),
// while the second correction's error is below (1/2 + 2^-22) beta 2^-24 ulp, which is
// smaller whenever beta <= 1 - 2^-20.  Steps with a significand above that, exponents
// outside [-60, 60] and zero points beyond 2^23 take the true division.
//
// That sequence is still 6 of the 13 operations an element costs, and it only matters next to a
// rounding tie.  So the common case is screened: q' = RN(a y + Z) in one FMA, n' = rint(q').
// With Q = a / Step, the value the definition rounds is v = RN(Q) + Z, and
//   |q' - v| <= |Q| 2^-23 + ulp(q') / 2  <=  (257 + |Z|) 2^-23 + 2^-16   wherever n' is in [-1, 256],
// so if q' is farther than delta = (258 + |Z|) 2^-23 + 2^-15 from every half-integer, v lies in
// the same unit interval and rint(RN(Q)) + Z = n' (outside [-1, 256] the relative error 2^-22
// keeps both on the same side of the clamp).  Units of 8 values with an element inside delta
// (about 1.5e-4 of all elements for |Z| <= 255) are redone with the exact sequence.  Binary32 input takes the screened
// quotient too, where |Z| allows it, and divides the units with a quotient beyond 2^22 (7419 x 4096 tokens x channels:
// 47.4 us with the division everywhere, 40.1 now; a quotient that underflows on the way rounds to 0 either way).
#include "act_unit.hpp"
#include "quant_act.hpp"
#include <type_traits>

namespace aweq {

typedef unsigned v2u __attribute__((ext_vector_type(2)));

constexpr int kQaBlock = 256;
constexpr int kQaWaves = kQaBlock / kWave;
constexpr int kQaVpt = 2;                               // panels (units per thread per row) per wavefront
constexpr int kQaPanels = kQaWaves * kQaVpt;            // 8 panels = 512 columns per block
constexpr int kQaMaxRows = 512;                         // rows per block (LDS row-sum slots)
constexpr int kQaSliceRows = 32;                        // slices are whole multiples of this
constexpr unsigned kQaXcds = 8;                         // workgroup id % 8 names the XCD a workgroup runs on

// One-dimensional grid over the (row slice, column chunk) pairs, column chunks of 8 panels varying fastest.
// Workgroup ids are dealt round-robin to the 8 XCDs, and the pass runs 12 - 23 % faster (K = 8192 / 4096;
// nothing to gain or lose at K = 22016) when each XCD works through a contiguous eighth of that sequence
// - a compact range of rows of X and of every output panel - instead of every eighth pair, so id b takes
// pair (b % 8) * ceil(pairs / 8) + b / 8.
// The codes go out in the K-panel layout the
// GEMM reads (64-byte panels, rows back to back), so a wavefront works on 8 rows x one panel
// per instruction: lane = 8 (row % 8) + unit; its load covers 8 whole 128-byte lines of
// binary16 input and its store 512 contiguous bytes of codes.  Each wavefront owns two
// panels, so a lane keeps the column sums of its 16 columns over the rows it visits.
// SUMS: neither codes nor row sums are asked for (a calibration without the forward): 14331 x 11008 binary16 72.3 -> 66.3 us
// without packing the codes, 7419 x 4096 binary32 29.5.
// KEEP: the codes are stored through the caches for the GEMM that reads them next (rule and figures at the launch).
// Whole groups of 8 rows x 2 whole panels of a wavefront go through a ring of two groups in flight, the first requested ahead of Step, Z and the
// scales, each refilled as soon as it has been consumed, and no load sits in a branch: with the loads predicated the compiler
// waited for all of them before every unit (us: sums alone 14331 x 11008 71 -> 60, 65536 x 4096 114 -> 102; codes and sums 8192 x 4096 34.1 -> 30.9,
// 16384 x 16384 175 -> 164, 5000 x 22016 95 -> 83; binary32 7419 x 4096 41.4 -> 36.5, 2048 x 512 10.5 -> 9.1; 262144 x 8192, at the memory's rate,
// 1178 -> 1174).  Four groups take 147 registers, three wavefronts to a SIMD: 63.0 / 32.7 / 158.6 in place of 59.7 / 30.8 / 163.4; one group
// 64 / 32 / 170.
// ADD: Step and Z come from the pieces of the range, and the sums go straight to their places, whole lines to an instruction: over tokens to one of
// `copies` rows, a row's, where several blocks have it, to rowsum_x (whole calibrations, us, partial rows and a merge -> this: 14331 x
// 11008 178.2 -> 177.2, 9000 x 4096 67.1 -> 64.2, 600 x 4096 with the forward 69.2 -> 66.6, 2000 x 16384 273 -> 262, 700 x 21888 108 -> 96.5,
// binary32 2048 x 512 28.1 -> 24.1).  A form of its own: with both in one kernel the other took up to 0.3 us more.
template <bool F16, bool SUMS, bool KEEP, bool ADD>
__global__ __launch_bounds__(kQaBlock) void quant_act_kernel(
    const void* __restrict__ X, int64_t T, int64_t K, int64_t ldx, const float* __restrict__ inv_s,
    const float* __restrict__ act_step, const int32_t* __restrict__ act_zero, int8_t* __restrict__ xq,
    int32_t* __restrict__ rowsum_x, int32_t* __restrict__ colsum_part, int rows_per_block, int chunks,
    unsigned pairs, uint32_t* status, RangeParts range, int copies)
{
    const unsigned pair = (blockIdx.x % kQaXcds) * (gridDim.x / kQaXcds) + blockIdx.x / kQaXcds;
    if (pair >= pairs) return;   // (the grid is rounded up to a multiple of 8)
    const int chunk = (int)(pair % (unsigned)chunks);
    const int64_t slice = pair / (unsigned)chunks;
    __shared__ int lds_rs[kQaMaxRows][kQaWaves];
    const int lane = threadIdx.x & (kWave - 1);
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x / kWave));
    const int rsub = lane >> 3, c8 = lane & 7;
    const int64_t r0 = slice * rows_per_block;
    const int nrows = (int)min((int64_t)rows_per_block, T - r0);
    const int64_t np = panel_count(K);

    const int64_t panel0 = (int64_t)chunk * kQaPanels + wave * kQaVpt;
    const int col0 = (int)(panel0 * kPanel) + c8 * 8;                      // K <= 2^31 - 1 columns
    int8_t* const dst0 = xq ? xq + (panel0 * T + r0) * kPanel + c8 * 8 : nullptr;   // this lane's 8 bytes of row r0, panel j = 0
    const int64_t dst_step = T * kPanel;                                   // to the next panel
    const char* const src0 = reinterpret_cast<const char*>(X) + (r0 * ldx + col0) * (F16 ? 2 : 4);
    bool valid[kQaVpt], pad[kQaVpt];
#pragma unroll
    for (int j = 0; j < kQaVpt; ++j) {
        valid[j] = col0 + j * kPanel < K;
        pad[j] = !valid[j] && panel0 + j < np;  // zero fill of the last panel
    }
    // Whole groups of 8 rows of whole panels go through a ring of kRing groups in flight, without a branch around any load: each
    // group's registers are refilled as soon as they have been consumed.  (With the loads predicated the compiler waited for all of
    // them before each unit.)
    constexpr int kRing = 2;
    const bool whole = (panel0 + kQaVpt) * kPanel <= K && nrows >= 8 * kRing;   // uniform in the wavefront
    const int ring_groups = whole ? nrows / (8 * kRing) * kRing : 0;
    RawUnit<F16> raw[kRing][kQaVpt];
    auto request = [&](int b, int group) {
#pragma unroll
        for (int j = 0; j < kQaVpt; ++j) raw[b][j].load(src0, (int64_t)(8 * group + rsub) * ldx + j * kPanel);
    };
    // binary16, any rows and columns (binary32 has no registers for it: 65536 x 64 11.1 -> 11.8 us)
    auto request_any = [&](int row) {
#pragma unroll
        for (int j = 0; j < kQaVpt; ++j)
            if (row < nrows && valid[j]) raw[0][j].load(src0, (int64_t)row * ldx + j * kPanel);
    };
    if (whole) {
#pragma unroll
        for (int b = 0; b < kRing; ++b) request(b, b);
    } else if (F16) {
        request_any(rsub);
    }

    uint32_t st = 0;
    float step;
    int zero;
    if constexpr (ADD) {   // Step and Z are not there yet: every block finds them, the first one stores them
        __shared__ float slot[2 * kQaWaves];
        const float2 r = parts_extremes<kQaBlock>(range.ext, range.blocks, 2, slot);
        uint32_t range_st = 0;
        qparams(r.x, r.y, 8, step, zero, range_st);
        if (blockIdx.x == 0 && threadIdx.x == 0) {
            st = range_st;
            range.xhat_range[0] = r.x; range.xhat_range[1] = r.y;
            *range.act_step = step;
            *range.act_zero = zero;
        }
    } else {
        step = *act_step;
        zero = *act_zero;
    }
    const ActParams p = quot_params(step, zero);
    float is[kQaVpt][8];
    bool fast_thread = p.fast;
    float is_max = 0.0f;
#pragma unroll
    for (int j = 0; j < kQaVpt; ++j) {
        // (the last unit again past the edge; 16 bytes at a time, aligned to 4)
        typedef float v4f_ __attribute__((ext_vector_type(4), aligned(4)));
        const v4f_* const q = reinterpret_cast<const v4f_*>(inv_s + min((int64_t)col0 + j * kPanel, K - 8));
        const v4f_ a = q[0], b = q[1];
#pragma unroll
        for (int i = 0; i < 4; ++i) { is[j][i] = a[i]; is[j][4 + i] = b[i]; }
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            // the exactness argument needs a y not to overflow: binary16 |x| < 2^16, Step >= 2^-60
            if (!(fabsf(is[j][i]) < 1.0e12f)) fast_thread = false;
            is_max = fmaxf(is_max, fabsf(is[j][i]));
        }
    }
    // the screened path does not track the largest quotient: it needs |x inv_s / Step| < 2^24
    // for every binary16 x up front (65504 max|inv_s| / Step with a margin for the roundings)
    const bool screen_thread = fast_thread && p.screen && 65600.0f * is_max * p.rstep < 16777216.0f;
    // one path for the whole block (the choice is uniform unless an inv_s is absurd)
    const bool fast = F16 ? __syncthreads_and(fast_thread ? 1 : 0) != 0 : p.screen;
    const bool screen = F16 ? __syncthreads_and(screen_thread ? 1 : 0) != 0 : p.screen;
    float big = 0.0f;
    float csf[kQaVpt][8];
    int csi[kQaVpt][8];
#pragma unroll
    for (int j = 0; j < kQaVpt; ++j)
#pragma unroll
        for (int i = 0; i < 8; ++i) { csf[j][i] = 0.0f; csi[j][i] = 0; }
    int my_rows = 0;

    // one unit: its code bytes to d
    auto unit = [&](auto mode_c, const RawUnit<F16>& u, int j, int8_t* d, int& rs) {
        constexpr int MODE = decltype(mode_c)::value;
        float x[8];
        u.get(x);
        const uint2 w = act_unit<MODE, SUMS>(x, is[j], p, csf[j], csi[j], rs, big, st);
        if (!SUMS && d) {   // (sums only: no code buffer)
            if constexpr (KEEP) *reinterpret_cast<v2u*>(d) = v2u{w.x, w.y};
            else __builtin_nontemporal_store(v2u{w.x, w.y}, reinterpret_cast<v2u*>(d));
        }
    };
    auto row_sum = [&](int rs, int row, bool ok) {
        if constexpr (!SUMS) {
            rs = group_allreduce<3>(rs, OpAdd());  // the 8 lanes of one row
            if (ok && c8 == 0) lds_rs[row][wave] = rs;
        }
    };
    int first = 0;   // rows that the ring has taken
    auto ring = [&](auto mode_c) {
        auto take = [&](int b, int group) {
            const int row = 8 * group + rsub;
            int rs = 0;
#pragma unroll
            for (int j = 0; j < kQaVpt; ++j) unit(mode_c, raw[b][j], j, dst0 ? dst0 + j * dst_step + row * kPanel : nullptr, rs);
            row_sum(rs, row, true);
        };
        int g = 0;
        for (; g + kRing < ring_groups; g += kRing) {
#pragma unroll
            for (int b = 0; b < kRing; ++b) { take(b, g + b); request(b, g + kRing + b); }
        }
#pragma unroll
        for (int b = 0; b < kRing; ++b) take(b, g + b);
        my_rows += ring_groups;
        first = 8 * ring_groups;
    };
    // any rows and columns, one group of 8 rows at a time, binary16 with the next one on its way (20000 x 120 7.8 -> 6.9 us)
    auto rest = [&](auto mode_c) {
        if (F16 && first > 0) request_any(first + rsub);
#pragma unroll 1
        for (int rb = first; rb < nrows; rb += 8) {
            const int row = rb + rsub;
            const bool row_ok = row < nrows;
            if (!F16) request_any(row);
            RawUnit<F16> u[kQaVpt];
#pragma unroll
            for (int j = 0; j < kQaVpt; ++j) u[j] = raw[0][j];
            if (F16) request_any(row + 8);
            int rs = 0;
            if (row_ok) {
                ++my_rows;
#pragma unroll
                for (int j = 0; j < kQaVpt; ++j) {
                    int8_t* const d = dst0 ? dst0 + j * dst_step + row * kPanel : nullptr;
                    if (valid[j]) unit(mode_c, u[j], j, d, rs);
                    else if (pad[j] && d) *reinterpret_cast<uint2*>(d) = make_uint2(0u, 0u);
                }
            }
            row_sum(rs, row, row_ok);
        }
    };
    // Whole groups one at a time, the next one on its way, for |Z| beyond the screen: its quotient takes the registers of the second group,
    // and more would cost a wavefront everywhere (us, Z = 6000, 16384 x 11008, one group requested once the last was done -> this: codes and
    // sums 134 -> 115, codes 132 -> 114, sums alone 100 -> 80).
    auto whole_rows = [&](auto mode_c) {
#pragma unroll 1
        for (int g = 0; g < ring_groups; ++g) {
            RawUnit<F16> u[kQaVpt];
#pragma unroll
            for (int j = 0; j < kQaVpt; ++j) u[j] = raw[0][j];
            request(0, min(g + 1, ring_groups - 1));
            const int row = 8 * g + rsub;
            int rs = 0;
#pragma unroll
            for (int j = 0; j < kQaVpt; ++j) unit(mode_c, u[j], j, dst0 ? dst0 + j * dst_step + row * kPanel : nullptr, rs);
            row_sum(rs, row, true);
        }
        my_rows += ring_groups;
        first = 8 * ring_groups;
    };
    if constexpr (F16) {
        if (screen) {
            if (whole) ring(std::integral_constant<int, 2>{});
            rest(std::integral_constant<int, 2>{});
        } else if (fast) {
            if (whole) whole_rows(std::integral_constant<int, 1>{});
            rest(std::integral_constant<int, 1>{});
        }
        else rest(std::integral_constant<int, 0>{});
    } else {
        if (screen) {
            if (whole) ring(std::integral_constant<int, 3>{});
            rest(std::integral_constant<int, 3>{});
        } else rest(std::integral_constant<int, 0>{});
    }
    if (big >= 16777216.0f) st |= AWEQ_ST_BIGQUOT;
    raise_status(status, st);

    if (colsum_part) {
        // lanes l, l ^ 8, l ^ 16, l ^ 32 hold the same columns for different rows; this block's sums over
        // its row slice (at most 512 rows of codes in [-128, 127]) go to row `slice` of the partial buffer, or are added to one of `copies` rows
        int32_t* const part = colsum_part + (ADD ? (int)(slice % copies) : slice) * K;
#pragma unroll
        for (int j = 0; j < kQaVpt; ++j) {
            int v[8];
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                v[i] = fast ? ((int)csf[j][i] - 128 * my_rows) : csi[j][i];
                v[i] += xor8(v[i]);
                v[i] += partner<4>(v[i]);
                v[i] += partner<5>(v[i]);
            }
            if constexpr (ADD) {
                // (a wavefront's 64 neighbouring columns in one instruction: lane l the column l / 8 of the eight that unit l % 8 has)
                int own = v[0];
#pragma unroll
                for (int i = 1; i < 8; ++i) own = rsub == i ? v[i] : own;
                if (valid[j]) atomicAdd(part + col0 + j * kPanel + rsub, own);
            } else if (lane < 8 && valid[j]) {
                typedef int v4i_ __attribute__((ext_vector_type(4)));
                v4i_* d = reinterpret_cast<v4i_*>(part + col0 + j * kPanel);
                d[0] = v4i_{v[0], v[1], v[2], v[3]};
                d[1] = v4i_{v[4], v[5], v[6], v[7]};
            }
        }
    }
    if constexpr (SUMS) return;
    __syncthreads();
    // with several column chunks `rowsum_x` is the partial buffer [chunks][T], folded by the merge kernel, or is added to
    if (rowsum_x)
        for (int i = threadIdx.x; i < nrows; i += kQaBlock) {
            int tot = 0;
#pragma unroll
            for (int w = 0; w < kQaWaves; ++w) tot += lds_rs[i][w];
            if (ADD && chunks > 1) atomicAdd(rowsum_x + r0 + i, tot);
            else rowsum_x[(int64_t)chunk * T + r0 + i] = tot;
        }
}

// Fold the per-slice column sums (fixed order, 64-bit) and the per-chunk row sums.  Blocks
// [0, col_blocks) own 32 columns each: 32 groups of 32 threads take every 32nd slice (few dependent loads
// per thread: the kernel is bound by their latency) and meet in LDS; the remaining blocks own 1024 rows each.
constexpr int kQaMergeCols = 32, kQaMergeParts = 32;
__global__ __launch_bounds__(kQaMergeCols * kQaMergeParts) void quant_act_merge(
    const int32_t* __restrict__ colsum_part, int slices, int64_t K, long long* __restrict__ colsum_xq,
    const int32_t* __restrict__ rowsum_part, int chunks, int64_t T, int32_t* __restrict__ rowsum_x, int col_blocks)
{
    if ((int)blockIdx.x < col_blocks) {
        __shared__ long long s_s[kQaMergeParts][kQaMergeCols];
        const int c = threadIdx.x & (kQaMergeCols - 1), part = threadIdx.x / kQaMergeCols;
        const int64_t k = (int64_t)blockIdx.x * kQaMergeCols + c;
        long long s = 0;
        if (k < K)
            for (int j = part; j < slices; j += kQaMergeParts) s += colsum_part[(int64_t)j * K + k];
        s_s[part][c] = s;
        __syncthreads();
        if (part != 0) return;
#pragma unroll
        for (int q = 1; q < kQaMergeParts; ++q) s += s_s[q][c];
        if (k < K) colsum_xq[k] = s;
    } else {
        const int64_t t = ((int64_t)blockIdx.x - col_blocks) * (kQaMergeCols * kQaMergeParts) + threadIdx.x;
        if (t >= T) return;
        int tot = 0;
        for (int c = 0; c < chunks; ++c) tot += rowsum_part[(int64_t)c * T + t];
        rowsum_x[t] = tot;
    }
}

// ---- row form: a block owns ROWS whole rows, so their code sums are complete inside it and no partial buffer or merge
// is needed.  For calls that do not ask for column sums (a forward with a calibrated scale).  Small calls are bound by
// the launch and the round trips to memory: one launch instead of two (the figures are at the dispatch below), and a row's
// next unit is requested while this one is quantised, without a branch around the load (3000 x 4104 14.7 -> 12.6 us, 4096 x 4096 15.2 -> 14.1; with the stores that stay in the caches, whole int8 forward, us:
// 300 tokens 4096 x 11008 46.4 -> 40.5, 2048 tokens 99.2 -> 95.6, 4096 tokens 11008 x 4096 182.6 -> 178.6).
constexpr int kQrBlock = 512;
template <bool F16, int ROWS>
__global__ __launch_bounds__(kQrBlock) void quant_act_rows(
    const void* __restrict__ X, int64_t T, int64_t K, int64_t ldx, const float* __restrict__ inv_s,
    const float* __restrict__ act_step, const int32_t* __restrict__ act_zero, int8_t* __restrict__ xq,
    int32_t* __restrict__ rowsum_x, uint32_t* status)
{
    __shared__ int s_rs[kQrBlock / kWave][ROWS];
    const int64_t r0 = (int64_t)blockIdx.x * ROWS;
    const int nrows = (int)min((int64_t)ROWS, T - r0);
    const int64_t units = K / 8, padded = panel_count(K) * (kPanel / 8);
    // the first unit of every row is requested ahead of Step and Z, the next one as soon as a unit has been consumed (without a branch
    // around a load: past the end the last unit, the last row again, not stored)
    RawUnit<F16> raw[ROWS];
    Float4 isa, isb;
    auto request = [&](int i, int64_t u) { raw[i].load(X, (r0 + min(i, nrows - 1)) * ldx + min(u, units - 1) * 8); };
    auto request_is = [&](int64_t u) {
        const float* const q = inv_s + min(u, units - 1) * 8;
        isa = *reinterpret_cast<const Float4*>(q);
        isb = *reinterpret_cast<const Float4*>(q + 4);
    };
    if ((int64_t)(threadIdx.x & ~(kWave - 1u)) < units) {   // (short rows leave wavefronts without a unit: binary32 2048 x 1032 4.8 -> 4.45 us)
#pragma unroll
        for (int i = 0; i < ROWS; ++i) request(i, threadIdx.x);
    }
    request_is(threadIdx.x);
    const ActParams p = quot_params(*act_step, *act_zero);
    uint32_t st = 0;
    float big = 0.0f;
    int rs[ROWS];
#pragma unroll
    for (int i = 0; i < ROWS; ++i) rs[i] = 0;
    auto take = [&](int64_t u, auto more_c) {
        int8_t* const d = xq + ((u >> 3) * T + r0) * kPanel + (u & 7) * 8;
        float is[8];
#pragma unroll
        for (int i = 0; i < 4; ++i) { is[i] = isa.f[i]; is[4 + i] = isb.f[i]; }
        if constexpr (decltype(more_c)::value) request_is(u + kQrBlock);
#pragma unroll
        for (int i = 0; i < ROWS; ++i) {
            float x[8];
            raw[i].get(x);
            if constexpr (decltype(more_c)::value) request(i, u + kQrBlock);
            if (i >= nrows) continue;
            const uint2 w = act_unit_any<F16>(x, is, p, rs[i], big, st);
            *reinterpret_cast<v2u*>(d + i * kPanel) = v2u{w.x, w.y};
        }
    };
    int64_t u = threadIdx.x, base = 0;
    for (; base + kQrBlock < units; base += kQrBlock, u += kQrBlock) take(u, std::true_type{});   // (a whole block of units, and more to come)
    if (u < units) take(u, std::false_type{});
    else if (u < padded) {                     // zero fill of the last panel (a multiple of 8 units, like the blocks of them)
        int8_t* const d = xq + ((u >> 3) * T + r0) * kPanel + (u & 7) * 8;
        for (int i = 0; i < nrows; ++i) *reinterpret_cast<uint2*>(d + i * kPanel) = make_uint2(0u, 0u);
    }
    if (big >= 16777216.0f) st |= AWEQ_ST_BIGQUOT;
    raise_status(status, st);
    if (!rowsum_x) return;
#pragma unroll
    for (int i = 0; i < ROWS; ++i) {
        const int v = wave_allreduce(rs[i], OpAdd());
        if ((threadIdx.x & (kWave - 1)) == 0) s_rs[threadIdx.x / kWave][i] = v;
    }
    __syncthreads();
    if ((int)threadIdx.x < nrows) {
        int tot = 0;
#pragma unroll
        for (int w = 0; w < kQrBlock / kWave; ++w) tot += s_rs[w][threadIdx.x];
        rowsum_x[r0 + threadIdx.x] = tot;
    }
}

struct QaPlan {
    int chunks;      // column chunks of 8 panels
    int64_t slices;  // row slices
    int64_t rpb;     // rows per slice
};

static QaPlan qa_plan(int64_t T, int64_t K)
{
    QaPlan p;
    p.chunks = (int)cdiv(panel_count(K), kQaPanels);
    int64_t slices = cdiv(8192, p.chunks);
    int64_t rpb = cdiv(T, slices);
    rpb = cdiv(rpb, kQaSliceRows) * kQaSliceRows;
    if (rpb > kQaMaxRows) rpb = kQaMaxRows;
    p.rpb = rpb;
    p.slices = cdiv(T, rpb);
    return p;
}

// The launch's slices: as many blocks as are resident at a time, since every block begins with the same round trips (for Step, Z, the scales) before
// its rows stream; never more slices than qa_plan has, which sizes the workspace.  us, 8192 blocks -> about 1024: sums alone 14331 x 11008
// 60.3 -> 54.4, 8000 x 11008 47.6 -> 35.1, 20000 x 4096 46.7 -> 32.6, 65536 x 4096 102 -> 89; codes and sums 16384 x 4096 50.6 -> 42.0, 4000 x 11008
// 40.2 -> 36.4, but beyond 2^27 values 3072 (65536 x 4096: 161 with 8192, 141 with 3072, 149 with 1024); binary32 7419 x 4096 36.4 with 2048 or
// more, 38.5 with 1024.  added (no partial rows): calls of few blocks in slices of 16 rows, less than that and the blocks of a column wait for
// each other's additions (whole calibrations, us, slices of 32 / 16 / 8 rows: 512 x 4096 33.1 / 32.0, binary32 700 x 2048 32.6 / 30.9, 2048 x 512
// 25.4 / 25.4 / 27.4, but 256 blocks, 4000 x 1024, 38.7 / 40.4).
static QaPlan launch_plan(int64_t T, int64_t K, bool f16, bool sums, bool added)
{
    QaPlan p = qa_plan(T, K);
    const int64_t blocks = f16 && (sums || T * K <= (1ll << 27)) ? 1024 : 3072;
    int64_t rpb = cdiv(cdiv(T, cdiv(blocks, p.chunks)), kQaSliceRows) * kQaSliceRows;
    if (rpb > kQaMaxRows) rpb = kQaMaxRows;
    if (rpb > p.rpb) p.rpb = rpb;
    if (added && p.rpb == kQaSliceRows && cdiv(T, kQaSliceRows) * p.chunks <= 128) p.rpb = kQaSliceRows / 2;
    p.slices = cdiv(T, p.rpb);
    return p;
}

bool quant_act_adds_rows(int64_t K) { return panel_count(K) > kQaPanels; }

// workspace: per-slice column sums [slices][K] int32, then (several column chunks only) per-chunk
// row sums [chunks][T] int32
size_t quant_act_ws_bytes(int64_t T, int64_t K)
{
    const QaPlan p = qa_plan(T, K);
    return (size_t)p.slices * (size_t)K * 4 + (p.chunks > 1 ? (size_t)p.chunks * (size_t)T * 4 : 0);
}

int launch_quant_act(const void* X, aweq_dtype dt, int64_t T, int64_t K, int64_t ldx, const float* inv_s,
                     const float* act_step, const int32_t* act_zero, int8_t* xq, int32_t* rowsum_x,
                     int64_t* colsum_xq, void* ws, uint32_t* status, hipStream_t st, const RangeParts* range,
                     int32_t* colsum_added, int copies)
{
    // Whole rows per block where nothing is summed over tokens, up to the size where the panel form streams as fast (us, panel form -> row
    // form: K = 4096: 1000 tokens 11.2 -> 6.4, 4096: 17.9 -> 14.1, 16384: 41.3 -> 40.1, but 32768: 74.0 -> 81.6; K = 11008: 2048 tokens 24.4 -> 17.8,
    // 8192: 58.6 -> 57.9, but 16384: 100 -> 107; 8192 x 22016 106 -> 109; binary32 16000 x 4096 68.7 -> 64.5, 5000 x 11008 63.7 -> 56.8).  Narrow
    // rows leave part of a block idle: 4097 x 1032 11.6 -> 9.5, but 8192 x 1032 13.2 -> 15.2.  One row per block
    // up to 256 tokens, two up to 1536, 768 blocks, three a compute unit, in place of 384 (4 / 2 rows: 1030 x 4096 5.8 / 5.0, 1536 x 4096 6.75 / 5.9,
    // 1536 x 11008 15.6 / 13.5, binary32 1500 x 4096 7.9 / 7.0, but 1700 x 4096 6.95 / 7.05; 1 / 2 rows: 600 x 4096 4.3 / 4.25).  Rows of up to 512 columns, one chunk of the panel
    // form, which then needs no merge: up to 2048 tokens where a row's sum is asked for (K = 64 / 512, 2048 tokens 5.5 -> 4.8 / 7.3 -> 4.9,
    // 2500 tokens 5.6 -> 7.0 / 7.3 -> 7.1, binary32 4096 tokens 5.3 -> 7.6 / 8.4 -> 9.9;
    // without the sums 2758 tokens K = 448 6.3 -> 4.8, 4051 tokens K = 120 5.9 -> 5.2).  Not where an output lies over what other
    // blocks still read: the panel form's merge writes the row sums in a launch of its own, and its blocks have 32 rows or more.
    const int64_t rows_most = rowsum_x && K <= kQaPanels * kPanel ? 2048 : K < 2048 ? 4096 : T * K <= (6ll << 24) ? 16384 : 4096;
    if (!range && !colsum_xq && xq && aligned16(inv_s) && T <= rows_most &&
        !overlap({{rowsum_x, T * 4}, {xq, T * panel_count(K) * kPanel}}, {matrix_span(X, T, K, ldx, dtype_size(dt)), {inv_s, K * 4}, {act_step, 4}, {act_zero, 4}})) {
#define AWEQ_QR(F, R) quant_act_rows<F, R><<<(unsigned)cdiv(T, R), kQrBlock, 0, st>>>(X, T, K, ldx, inv_s, act_step, act_zero, xq, rowsum_x, status)
        if (dt == AWEQ_F16) { if (T <= 256) AWEQ_QR(true, 1); else if (T <= 1536) AWEQ_QR(true, 2); else AWEQ_QR(true, 4); }
        else { if (T <= 256) AWEQ_QR(false, 1); else if (T <= 1536) AWEQ_QR(false, 2); else AWEQ_QR(false, 4); }
#undef AWEQ_QR
        return launch_status();
    }
    const bool sums = !xq && !rowsum_x;
    const QaPlan p = launch_plan(T, K, dt == AWEQ_F16, sums, colsum_added != nullptr);
    if (p.slices * p.chunks > 0x7ffffff0ll) return AWEQ_ERR_SHAPE;
    const bool multi = p.chunks > 1;
    int32_t* const colsum_part = colsum_added ? colsum_added : colsum_xq ? reinterpret_cast<int32_t*>(ws) : nullptr;
    int32_t* const rowsum_part = reinterpret_cast<int32_t*>(ws) + (size_t)p.slices * K;
    int32_t* const rs_out = !rowsum_x ? nullptr : (multi && !colsum_added ? rowsum_part : rowsum_x);
    const unsigned pairs = (unsigned)(p.slices * p.chunks);
    const unsigned grid = (unsigned)(cdiv(pairs, kQaXcds) * kQaXcds);
    const RangeParts parts = range ? *range : RangeParts{};   // (with colsum_added only)
    // codes that fit the memory-side cache are stored through the caches, where the GEMM finds them; more would only evict each
    // other (int8 forward, us, non-temporal -> cached: 16384 tokens 4096 x 11008 (180 MB) 663 -> 650, 4096 x 16384 (268 MB)
    // 979 -> 967, 12000 tokens 8192 x 16384 1306 -> 1307; the pass alone at 262144 x 8192 (2.1 GB) 1188 -> 1268)
    const bool keep = xq && (int64_t)panel_count(K) * kPanel * T <= kCacheBytes;
#define AWEQ_QA(F, S, P, A) quant_act_kernel<F, S, P, A><<<grid, kQaBlock, 0, st>>>(X, T, K, ldx, inv_s, act_step, act_zero, xq, rs_out, colsum_part, (int)p.rpb, p.chunks, pairs, status, parts, copies)
#define AWEQ_QF(F, A) do { if (sums) AWEQ_QA(F, true, false, A); else if (keep) AWEQ_QA(F, false, true, A); else AWEQ_QA(F, false, false, A); } while (0)
    if (colsum_added) { if (dt == AWEQ_F16) AWEQ_QF(true, true); else AWEQ_QF(false, true); }
    else { if (dt == AWEQ_F16) AWEQ_QF(true, false); else AWEQ_QF(false, false); }
#undef AWEQ_QF
#undef AWEQ_QA
    if (colsum_added) return launch_status();
    const int col_blocks = colsum_xq ? (int)cdiv(K, kQaMergeCols) : 0;
    const int64_t row_blocks = (rowsum_x && multi) ? cdiv(T, kQaMergeCols * kQaMergeParts) : 0;
    if (col_blocks + row_blocks > 0)
        quant_act_merge<<<(unsigned)(col_blocks + row_blocks), kQaMergeCols * kQaMergeParts, 0, st>>>(
            colsum_part, (int)p.slices, K, reinterpret_cast<long long*>(colsum_xq), rowsum_part, p.chunks, T, rowsum_x, col_blocks);
    return launch_status();
}

int check_quant_act_args(const void* X, aweq_dtype dt, int64_t T, int64_t K, int64_t ldx, const float* inv_s,
                         const float* act_step, const int32_t* act_zero, const int8_t* xq, bool xq_optional)
{
    if (!X || !inv_s || !act_step || !act_zero || (!xq && !xq_optional)) return AWEQ_ERR_NULL;
    if (dt != AWEQ_F32 && dt != AWEQ_F16) return AWEQ_ERR_DTYPE;
    if (T <= 0 || K <= 0 || ldx < K || (K % 8) != 0) return AWEQ_ERR_SHAPE;
    if (!aligned16(X) || ((size_t)ldx * dtype_size(dt)) % 16 != 0 || !aligned16(xq)) return AWEQ_ERR_ALIGN;
    return AWEQ_OK;
}

// the sums need the workspace (rowsum_x only with several column chunks)
int check_quant_act_ws(int64_t T, int64_t K, const int32_t* rowsum_x, const int64_t* colsum_xq, const void* ws, size_t ws_bytes)
{
    const bool need = colsum_xq || (rowsum_x && qa_plan(T, K).chunks > 1);
    if (!need) return AWEQ_OK;
    if (!ws || ws_bytes < quant_act_ws_bytes(T, K)) return AWEQ_ERR_WORKSPACE;
    if (!aligned16(ws)) return AWEQ_ERR_ALIGN;
    return AWEQ_OK;
}

}  // namespace aweq

using namespace aweq;

extern "C" int aweq_quant_act(const void* X, aweq_dtype dt, int64_t T, int64_t K, int64_t ldx,
                              const float* inv_s, const float* act_step, const int32_t* act_zero,
                              int8_t* xq, int32_t* rowsum_x, int64_t* colsum_xq,
                              void* ws, size_t ws_bytes, uint32_t* status, void* stream)
{
    if (!xq && !rowsum_x && !colsum_xq) return AWEQ_ERR_NULL;   // nothing to produce
    int rc = check_quant_act_args(X, dt, T, K, ldx, inv_s, act_step, act_zero, xq, true);
    if (rc != AWEQ_OK) return rc;
    rc = check_quant_act_ws(T, K, rowsum_x, colsum_xq, ws, ws_bytes);
    if (rc != AWEQ_OK) return rc;
    return launch_quant_act(X, dt, T, K, ldx, inv_s, act_step, act_zero, xq, rowsum_x, colsum_xq, ws, status, as_stream(stream));
}
