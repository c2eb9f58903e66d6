// Stages 2b, 3 and 5 of a calibration in one pass over each weight: W_hat = W s (Eq. 3), its codes (Eq. 1-2) and the bias correction
// (Sec. 3.3, Eq. 11-15), W read once and neither W_hat nor the codes read back: 2 + 2 + 1 bytes (8 bits) or 2 + 2 + 1/2 (4 bits) an element of
// binary16, where the three stages one after the other move 8 / 7.  Bound by its vector operations: with all its stores left out a calibration of 14331
// tokens 4096 x 11008 took 166 us instead of 178.
//
// A block (a wavefront of short rows) takes one to four output channels at a time, so that what every channel needs of a column is read and
// prepared as much less often (s and E[x_hat], 8 bytes; for 8 bits also the sum of the activation codes, 4 bytes a copy, whose digits are formed here: 12
// bytes, with four copies of a narrow matrix's sums 24), and keeps the rows in registers between the extremes and the codes.
//
// The sums over tokens that the int8 path's correction needs are the column sums of the activation codes times the weight codes:
// sum_t acc[t,n] = sum_k wq[n,k] colsum_xq[k], the same integers that a GEMM adds up.
#include "weight_pass.hpp"
#include "code_digits.hpp"
#include "row_reduce.hpp"
#include "weight_unit.hpp"

namespace aweq {

constexpr int kPassRows = 4;

template <int NT>
__device__ __forceinline__ void finish_ranges(const FinishArgs& f, int64_t K, unsigned block, int copies)
{
    __shared__ float slot[3][2 * (NT / kWave)];
    const float2 x = parts_extremes<NT>(f.range.ext, f.range.blocks, 0, slot[0]);
    const float2 w = parts_extremes<NT>(f.range.ext, f.range.blocks, 1, slot[1]);
    const float Rx = (x.y - x.x) + 0.0f, Rw = (w.y - w.x) + 0.0f;   // (a tensor of zeros of both signs has range +0)
    const int64_t k = (int64_t)block * NT + threadIdx.x;
    if (k < K) {
        if (f.p_x) f.p_x[k] = f.r_x[k] / Rx;
        if (f.p_w) f.p_w[k] = f.r_w[k] / Rw;
        if (f.colsum) {
            int c = f.colsum[k];
            for (int64_t j = K; j < copies * K; j += K) c += f.colsum[j + k];
            f.colsum_xq[k] = c;
        }
    }
    if (block != 0) return;
    if (threadIdx.x == 0) { *f.R_x = Rx; *f.R_w = Rw; }
    if (!f.range.act_step) return;
    const float2 h = parts_extremes<NT>(f.range.ext, f.range.blocks, 2, slot[2]);
    if (threadIdx.x == 0) {
        uint32_t st = 0;
        float step;
        int zero;
        qparams(h.x, h.y, 8, step, zero, st);
        f.range.xhat_range[0] = h.x; f.range.xhat_range[1] = h.y;
        *f.range.act_step = step;
        *f.range.act_zero = zero;
        raise_status(f.status, st);
    }
}

constexpr int kFinishThreads = 256;
__global__ __launch_bounds__(kFinishThreads) void calib_finish(FinishArgs f, int64_t K) { finish_ranges<kFinishThreads>(f, K, blockIdx.x, 1); }

__device__ __forceinline__ const PassMember& member_of(const PassArgs& a)
{
    int i = 0;
    while (i + 1 < a.n && blockIdx.x >= a.m[i + 1].first_block) ++i;
    return a.m[i];
}

// the parameters that lane `lane` holds, for every lane
__device__ __forceinline__ ActParams params_of_lane(const ActParams& v, int lane)
{
    auto f = [&](float x) { return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(x), lane)); };
    ActParams p = v;
    p.step = f(v.step);
    p.rstep = f(v.rstep);
    p.thr = f(v.thr);
    p.zero = __builtin_amdgcn_readlane(v.zero, lane);
    p.screen = __builtin_amdgcn_readlane(v.screen ? 1 : 0, lane) != 0;
    return p;
}
// the parameters that lane Q of each quad holds, for the four of them
template <int Q>
__device__ __forceinline__ ActParams params_of_quad(const ActParams& v)
{
    constexpr int ctrl = Q * 0x55;   // quad_perm [Q, Q, Q, Q]
    auto f = [&](float x) { return __int_as_float(dpp_mov<ctrl>(__float_as_int(x))); };
    ActParams p = v;
    p.step = f(v.step);
    p.rstep = f(v.rstep);
    p.thr = f(v.thr);
    p.zero = dpp_mov<ctrl>(v.zero);
    p.screen = dpp_mov<ctrl>(v.screen ? 1 : 0) != 0;
    return p;
}

template <bool F16>
__device__ __forceinline__ const void* row_at(const void* M, int64_t n, int64_t ld)
{
    return reinterpret_cast<const char*>(M) + (size_t)n * ld * (F16 ? 2 : 4);
}

// LINES: binary16 rows that are whole 128-byte lines, read for the last time and written for a later call: non-temporal both (figures at
// the launch; a line that two rows share would be fetched twice)
template <bool LINES, bool F16>
__device__ __forceinline__ void load_unit(Unit<F16>& u, const void* row, int64_t i)
{
    if constexpr (LINES) {
        typedef int v4i_ __attribute__((ext_vector_type(4)));
        u.raw = __builtin_bit_cast(Half8, __builtin_nontemporal_load(reinterpret_cast<const v4i_*>(reinterpret_cast<const _Float16*>(row) + i * 8)));
    } else {
        u.load(row, i);
    }
}
template <bool LINES, bool F16>
__device__ __forceinline__ void store_unit(const Unit<F16>& u, void* row, int64_t i)
{
    if constexpr (LINES) {
        typedef int v4i_ __attribute__((ext_vector_type(4)));
        __builtin_nontemporal_store(__builtin_bit_cast(v4i_, u.raw), reinterpret_cast<v4i_*>(reinterpret_cast<_Float16*>(row) + i * 8));
    } else {
        u.store(row, i);
    }
}

// x = RN(x s) to the weight's type (Eq. 3)
template <bool F16>
__device__ __forceinline__ void fold_unit(Unit<F16>& u, const Float4& s0, const Float4& s1)
{
    float x[8];
    u.get(x);
#pragma unroll
    for (int i = 0; i < 4; ++i) { x[i] = rounded_f32(x[i] * s0.f[i]); x[4 + i] = rounded_f32(x[4 + i] * s1.f[i]); }
    u.set(x);
}

// Extremes of a lane's elements of one row.  Binary16: two pairs to an operation, which hands a NaN on; then they are taken again without it.
// (With a minimum, a maximum and a test for NaN of every pair, and every lane's own elements held against Step, it had two operations an element
// more, and the pass is bound by its vector operations: us, whole calibrations, before -> this: 1000 tokens 11008 x 4096 79.6 -> 76.2, 2000 tokens
// 4096 x 16384 259 -> 249, 20000 tokens 8192 x 8192 215 -> 211, INT4 65536 tokens 11008 x 4096 145.9 -> 142.7, INT3 2048 tokens 4096 x 11008
// 80.6 -> 76.9; the byte conversion that clamps among it.)
template <bool F16> struct LaneExtremes;
template <>
struct LaneExtremes<true> {
    f16x2 lo = {(_Float16)INFINITY, (_Float16)INFINITY}, hi = {(_Float16)-INFINITY, (_Float16)-INFINITY};
    __device__ __forceinline__ void add(const Unit<true>& u)
    {
#pragma unroll
        for (int i = 0; i < 4; i += 2) {
            lo = __builtin_elementwise_minimum(__builtin_elementwise_minimum(lo, u.raw.h[i]), u.raw.h[i + 1]);
            hi = __builtin_elementwise_maximum(__builtin_elementwise_maximum(hi, u.raw.h[i]), u.raw.h[i + 1]);
        }
    }
    __device__ __forceinline__ void add_numbers(const Unit<true>& u)
    {
#pragma unroll
        for (int i = 0; i < 4; ++i) { lo = hmin2(lo, u.raw.h[i]); hi = hmax2(hi, u.raw.h[i]); }
    }
};
template <>
struct LaneExtremes<false> {
    float lo = INFINITY, hi = -INFINITY, bad = 0.0f;
    __device__ __forceinline__ void add(const Unit<false>& u)
    {
        float x[8];
        u.get(x);
        minmax8(x, lo, hi);
#pragma unroll
        for (int i = 0; i < 8; ++i) bad = __builtin_fmaf(x[i], 0.0f, bad);   // 0, or NaN from then on
    }
    __device__ __forceinline__ void add_numbers(const Unit<false>&) {}
};
// a NaN among this lane's elements of any row (binary32: or an infinity; either way a longer path with the same results)
template <int ROWS>
__device__ __forceinline__ bool any_nan(const LaneExtremes<true> (&ex)[ROWS])
{
    f16x2 s = ex[0].lo;
#pragma unroll
    for (int r = 1; r < ROWS; ++r) s = __builtin_elementwise_minimum(s, ex[r].lo);
    return s.x != s.x || s.y != s.y;
}
template <int ROWS>
__device__ __forceinline__ bool any_nan(const LaneExtremes<false> (&ex)[ROWS])
{
    float s = ex[0].bad;
#pragma unroll
    for (int r = 1; r < ROWS; ++r) s += ex[r].bad;
    return s != s;
}
// Whether a row whose elements lie in `range` (numbers; no NaN beside them) may take the screened quotient
__device__ __forceinline__ bool may_screen(float2 range, const ActParams& p)
{
    return p.screen && fmaxf(fabsf(range.x), fabsf(range.y)) * p.rstep < 8388608.0f;
}

// lowest and highest element of row (lane % ROWS), over groups of 2^LEVELS lanes
template <int LEVELS, int ROWS>
__device__ __forceinline__ float2 rows_extremes(const LaneExtremes<true> (&ex)[ROWS])
{
    f16x2 v[ROWS];   // minimum, and the maximum negated: both in one packed operation
#pragma unroll
    for (int r = 0; r < ROWS; ++r) {
        const f16x2 a = {ex[r].lo.x, -ex[r].hi.x}, b = {ex[r].lo.y, -ex[r].hi.y};
        v[r] = hmin2(a, b);
    }
    const f16x2 m = reduce_rows<ROWS, LEVELS>(v, OpMinH());
    return make_float2((float)m.x, -(float)m.y);
}
template <int LEVELS, int ROWS>
__device__ __forceinline__ float2 rows_extremes(const LaneExtremes<false> (&ex)[ROWS])
{
    float lo[ROWS], hi[ROWS];
#pragma unroll
    for (int r = 0; r < ROWS; ++r) { lo[r] = ex[r].lo; hi[r] = ex[r].hi; }
    return make_float2(reduce_rows<ROWS, LEVELS>(lo, OpMin()), reduce_rows<ROWS, LEVELS>(hi, OpMax()));
}

// ---- 8 bits, one (Step, Z) per output channel.  TPR threads hold ROWS rows in UPT units a row and thread, all requested before the first
// is used.  Lane r of each wavefront forms the parameters of row r (three divisions once instead of ROWS times).
template <bool F16, bool LINES, int TPR, int UPT, int ROWS>
__global__ __launch_bounds__(TPR == kWave ? 256 : TPR, TPR == 512 && UPT == 3 ? 4 : 1) void weight_pass_rows(PassArgs a)
{
    constexpr int kThreads = TPR == kWave ? 256 : TPR, kSets = kThreads / TPR, kWaves = TPR / kWave;
    static_assert(kSets == 1 || kWaves == 1, "rows are reduced over a wavefront or over the block");
    if (blockIdx.x >= a.weight_blocks) { finish_ranges<kThreads>(a.fin, a.K, blockIdx.x - a.weight_blocks, a.copies); return; }
    const PassMember& m = member_of(a);
    __shared__ float2 slot_ex[kWaves][ROWS];
    __shared__ double slot_d[kWaves][ROWS];
    __shared__ long long slot_l[kWaves][ROWS];
    __shared__ int slot_i[kWaves][ROWS];
    __shared__ long long slot_t[kWaves];
    const int lane = threadIdx.x & (kWave - 1), wave = kWaves > 1 ? threadIdx.x / kWave : 0, tid = threadIdx.x % TPR;
    const int64_t n0 = ((int64_t)(blockIdx.x - m.first_block) * kSets + threadIdx.x / TPR) * ROWS;
    if (kSets > 1 && n0 >= m.N) return;   // (no barriers where wavefronts have rows of their own)
    const int rows = (int)min((int64_t)ROWS, m.N - n0);
    const int64_t units = a.K / 8;
    uint32_t st = 0;

    Unit<F16> reg[ROWS][UPT];   // (past the edge: the last row again, not stored)
#pragma unroll
    for (int j = 0; j < UPT; ++j) {
        const int64_t u = tid + (int64_t)j * TPR;
        if (u < units) {
#pragma unroll
            for (int r = 0; r < ROWS; ++r) load_unit<LINES>(reg[r][j], row_at<F16>(m.W, n0 + min(r, rows - 1), m.ldw), u);
        }
    }
    LaneExtremes<F16> ex[ROWS];
#pragma unroll
    for (int j = 0; j < UPT; ++j) {
        const int64_t u = tid + (int64_t)j * TPR;
        if (u < units) {
            const Float4 s0 = *reinterpret_cast<const Float4*>(a.s + u * 8), s1 = *reinterpret_cast<const Float4*>(a.s + u * 8 + 4);
#pragma unroll
            for (int r = 0; r < ROWS; ++r) {
                fold_unit<F16>(reg[r][j], s0, s1);
                if (r < rows) store_unit<LINES>(reg[r][j], const_cast<void*>(row_at<F16>(m.W_hat, n0 + r, m.ldwh)), u);
                ex[r].add(reg[r][j]);
            }
        }
    }
    const int lr = lane % ROWS;
    const bool nan = __any(any_nan(ex));
    if (F16 && nan) {
#pragma unroll
        for (int r = 0; r < ROWS; ++r) {
            ex[r] = LaneExtremes<F16>();
#pragma unroll
            for (int j = 0; j < UPT; ++j)
                if (tid + (int64_t)j * TPR < units) ex[r].add_numbers(reg[r][j]);
        }
    }
    float2 range = rows_extremes<6>(ex);
    if constexpr (kWaves > 1) {
        if (lane < ROWS) slot_ex[wave][lane] = range;
        __syncthreads();
#pragma unroll
        for (int w = 0; w < kWaves; ++w) { const float2 e = slot_ex[w][lr]; range.x = fminf(range.x, e.x); range.y = fmaxf(range.y, e.y); }
    }
    float my_step;
    int my_zero;
    qparams(range.x, range.y, 8, my_step, my_zero, st);
    if (wave == 0 && lane < rows) { m.step[n0 + lane] = my_step; m.zero[n0 + lane] = my_zero; }
    ActParams mine = quot_params(my_step, my_zero);
    mine.screen = !nan && may_screen(range, mine);
    ActParams p[ROWS];
#pragma unroll
    for (int r = 0; r < ROWS; ++r) p[r] = params_of_lane(mine, r);

    double acc[ROWS];
    int rs[ROWS], cd[ROWS][4], td[4] = {0, 0, 0, 0};
#pragma unroll
    for (int r = 0; r < ROWS; ++r) {
        acc[r] = 0.0;
        rs[r] = 0;
#pragma unroll
        for (int j = 0; j < 4; ++j) cd[r][j] = 0;
    }
#pragma unroll
    for (int j = 0; j < UPT; ++j) {
        const int64_t u = tid + (int64_t)j * TPR;
        if (u < units) {
            const Float4 m0 = *reinterpret_cast<const Float4*>(a.mu + u * 8), m1 = *reinterpret_cast<const Float4*>(a.mu + u * 8 + 4);
            int cx[2][4] = {};
#pragma unroll
            for (int q = 0; q < (TPR == kWave ? kMostCopies : 1); ++q) {   // (the launch has TPR = kWave up to kCopiesK columns)
                if (q > 0 && q >= a.copies) break;
                const int4 c0 = *reinterpret_cast<const int4*>(a.colsum + q * a.K + u * 8), c1 = *reinterpret_cast<const int4*>(a.colsum + q * a.K + u * 8 + 4);
                cx[0][0] += c0.x; cx[0][1] += c0.y; cx[0][2] += c0.z; cx[0][3] += c0.w;
                cx[1][0] += c1.x; cx[1][1] += c1.y; cx[1][2] += c1.z; cx[1][3] += c1.w;
            }
            uint32_t d[2][4];
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                pack_digits(cx[h], d[h]);
#pragma unroll
                for (int i = 0; i < 4; ++i) td[i] = __builtin_amdgcn_sdot4(0x01010101, (int)d[h][i], td[i], false);
            }
            const int64_t off = (u >> 3) * m.N * kPanel + (u & 7) * 8;   // unit u of row 0 in the K-panel layout
#pragma unroll
            for (int r = 0; r < ROWS; ++r) {
                float x[8];
                reg[r][j].get(x);
                uint32_t w0, w1;
                unit_words<8>(x, p[r], p[r].screen, w0, w1, st);
                if (r < rows) *reinterpret_cast<uint2*>(m.codes + off + (n0 + r) * kPanel) = make_uint2(w0, w1);
                rs[r] += unit_sum(w0, w1);
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    acc[r] = __builtin_fma((double)x[i], (double)m0.f[i], acc[r]);
                    acc[r] = __builtin_fma((double)x[4 + i], (double)m1.f[i], acc[r]);
                    cd[r][i] = __builtin_amdgcn_sdot4((int)w0, (int)d[0][i], cd[r][i], false);
                    cd[r][i] = __builtin_amdgcn_sdot4((int)w1, (int)d[1][i], cd[r][i], false);
                }
            }
        }
    }
    const int64_t pad = units + tid;   // columns past K in the last panel are zero
    if (pad < panel_count(a.K) * 8) {
        for (int r = 0; r < rows; ++r)
            *reinterpret_cast<uint2*>(m.codes + ((pad >> 3) * m.N + n0 + r) * kPanel + (pad & 7) * 8) = make_uint2(0u, 0u);
    }
    raise_status(a.status, st);

    // the row of this lane (lane % ROWS), summed over the wavefront, then over the block
    long long cv[ROWS];
#pragma unroll
    for (int r = 0; r < ROWS; ++r) cv[r] = digits_value(cd[r]);
    double a_r = reduce_rows<ROWS, 6>(acc, OpAdd());
    long long c_r = reduce_rows<ROWS, 6>(cv, OpAdd());
    int r_r = reduce_rows<ROWS, 6>(rs, OpAdd());
    long long tot = wave_allreduce(digits_value(td), OpAdd());   // sum of colsum_xq over the columns
    if constexpr (kWaves > 1) {
        if (lane == 0) slot_t[wave] = tot;
        if (lane < ROWS) { slot_d[wave][lane] = a_r; slot_l[wave][lane] = c_r; slot_i[wave][lane] = r_r; }
        __syncthreads();
        if (wave != 0) return;
        a_r = 0.0; c_r = 0; r_r = 0; tot = 0;
#pragma unroll
        for (int w = 0; w < kWaves; ++w) {
            a_r += slot_d[w][lr];
            c_r += slot_l[w][lr];
            r_r += slot_i[w][lr];
            tot += slot_t[w];
        }
    }
    if (lane >= rows) return;
    const int64_t n = n0 + lane;
    const double d = int8_delta(a_r, c_r, r_r, tot, a.count, a.K, *a.act_step, *a.act_zero, my_step, my_zero);
    m.delta[n] = (float)d;
    m.bias_out[n] = (float)((m.bias_in ? (double)m.bias_in[n] : 0.0) + (a.enable_bc ? d : 0.0));
    if (m.rowsum) m.rowsum[n] = r_r;
    if (m.colsum_acc) m.colsum_acc[n] = c_r;
}

// ---- 4 / 3 bits, one (Step, Z) per group of 8 * 2^LEVELS consecutive k inside a row; weight-only correction (Eq. 12-15):
// delta = -sum_k (W~ - W_hat) E[x_hat].  A lane has the same unit of a group in four rows; lane q of each quad forms the parameters of row
// q (three divisions once instead of four times).  A block of BLOCK threads walks down its rows.  (Two units a lane, groups of 128, us:
// 11008 x 4096 47.8 -> 53.5, 22016 x 8192 163 -> 180: they take 197 registers, half the wavefronts.)
template <bool F16, bool LINES, int BITS, int LEVELS, int BLOCK>
__global__ __launch_bounds__(BLOCK, BLOCK == kWave ? 3 : 4) void weight_pass_groups(PassArgs a)
{
    constexpr int ROWS = kPassRows, kLanes = 1 << LEVELS, kWaves = BLOCK / kWave;
    static_assert(ROWS == 4 && LEVELS >= 2, "a quad lies inside a group");
    if (blockIdx.x >= a.weight_blocks) { finish_ranges<BLOCK>(a.fin, a.K, blockIdx.x - a.weight_blocks, 1); return; }
    const PassMember& m = member_of(a);
    __shared__ double slot_d[kWaves][ROWS];
    const int64_t n0 = (int64_t)(blockIdx.x - m.first_block) * ROWS;
    const int rows = (int)min((int64_t)ROWS, m.N - n0);
    const int64_t units = a.K / 8, row_bytes = a.K / 8 * BITS;
    uint32_t st = 0;
    double acc[ROWS];
#pragma unroll
    for (int r = 0; r < ROWS; ++r) acc[r] = 0.0;
    for (int64_t u = threadIdx.x; u < units; u += BLOCK) {   // (K % group == 0: a group is entirely in or out)
        Unit<F16> reg[ROWS];
#pragma unroll
        for (int r = 0; r < ROWS; ++r) load_unit<LINES>(reg[r], row_at<F16>(m.W, n0 + min(r, rows - 1), m.ldw), u);   // (past the edge: the last row again, not stored)
        const Float4 s0 = *reinterpret_cast<const Float4*>(a.s + u * 8), s1 = *reinterpret_cast<const Float4*>(a.s + u * 8 + 4);
        LaneExtremes<F16> ex[ROWS];
#pragma unroll
        for (int r = 0; r < ROWS; ++r) {
            fold_unit<F16>(reg[r], s0, s1);
            if (r < rows) store_unit<LINES>(reg[r], const_cast<void*>(row_at<F16>(m.W_hat, n0 + r, m.ldwh)), u);
            ex[r].add(reg[r]);
        }
        const bool nan = __any(any_nan(ex));
        if (F16 && nan) {
#pragma unroll
            for (int r = 0; r < ROWS; ++r) { ex[r] = LaneExtremes<F16>(); ex[r].add_numbers(reg[r]); }
        }
        const float2 range = rows_extremes<LEVELS>(ex);   // of row (lane % 4)
        float my_step;
        int my_zero;
        qparams(range.x, range.y, BITS, my_step, my_zero, st);
        const int in_group = (int)u & (kLanes - 1);
        if (in_group < rows) {   // (lanes 0 .. 3 of the group: rows 0 .. 3)
            const int64_t gi = (n0 + in_group) * (units >> LEVELS) + (u >> LEVELS);
            m.step[gi] = my_step;
            m.zero[gi] = my_zero;
        }
        ActParams mine = quot_params(my_step, my_zero);
        mine.screen = !nan && may_screen(range, mine);
        const ActParams p[ROWS] = {params_of_quad<0>(mine), params_of_quad<1>(mine), params_of_quad<2>(mine), params_of_quad<3>(mine)};
        const Float4 m0 = *reinterpret_cast<const Float4*>(a.mu + u * 8), m1 = *reinterpret_cast<const Float4*>(a.mu + u * 8 + 4);
#pragma unroll
        for (int r = 0; r < ROWS; ++r) {
            const bool screened = __all(p[r].screen);
            float x[8], diff[8];
            reg[r].get(x);
            uint32_t w0, w1;
            unit_words<BITS, true>(x, p[r], screened, w0, w1, st, diff);
            if (r < rows) store_unit_words<BITS>(w0, w1, m.codes + (n0 + r) * row_bytes, u);
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                const float wt = diff[i] * p[r].step;
                acc[r] = __builtin_fma((double)wt - (double)x[i], (double)(i < 4 ? m0.f[i] : m1.f[i - 4]), acc[r]);
            }
        }
    }
    raise_status(a.status, st);
    const double sum = reduce_rows<ROWS, 6>(acc, OpAdd());
    if (threadIdx.x % kWave < ROWS) slot_d[threadIdx.x / kWave][threadIdx.x % kWave] = sum;
    __syncthreads();
    if ((int)threadIdx.x >= rows) return;
    const int64_t n = n0 + threadIdx.x;
    double v = 0.0;
#pragma unroll
    for (int w = 0; w < kWaves; ++w) v += slot_d[w][threadIdx.x];
    const double d = -v;
    m.delta[n] = (float)d;
    m.bias_out[n] = (float)((m.bias_in ? (double)m.bias_in[n] : 0.0) + (a.enable_bc ? d : 0.0));
}

constexpr int64_t kPassK = 24576;   // columns whose rows fit a block's registers

bool weight_pass_takes(int bits, int group, bool w8a8, int64_t N, int64_t K, uint64_t count)
{
    if (N > (1ll << 30)) return false;
    if (w8a8)   // four signed digits hold column sums of |codes| <= 128 of fewer than 2^23 tokens
        return bits == 8 && group == 0 && K <= kPassK && count < (1ull << 23);
    return (bits == 4 || bits == 3) && (group == 32 || group == 64 || group == 128 || group == 256 || group == 512) && K % group == 0 &&
           N <= 65535 && K < (1ll << 26);   // (as aweq_quant_weight)
}

// blocks of `rows_per_block` rows for every member, then the ones of `fin`
static unsigned place_blocks(PassArgs& a, int rows_per_block, int threads)
{
    unsigned b = 0;
    for (int i = 0; i < a.n; ++i) {
        a.m[i].first_block = b;
        b += (unsigned)cdiv(a.m[i].N, rows_per_block);
    }
    a.weight_blocks = b;
    return b + (unsigned)cdiv(a.K, threads);
}

template <bool F16, bool LINES, int TPR, int UPT, int ROWS>
static void launch_rows(PassArgs& a, hipStream_t st)
{
    constexpr int threads = TPR == kWave ? 256 : TPR;
    weight_pass_rows<F16, LINES, TPR, UPT, ROWS><<<place_blocks(a, threads / TPR * ROWS, threads), threads, 0, st>>>(a);
}

// Threads x units x rows of a block (us with the launch, W found in the memory-side cache where it fits): few registers, so that several
// blocks of a compute unit are in different phases, and as many rows as those allow.  Binary16: 12288 x 4096 256 x 2 x 4 52.3, x 2 rows 53.0,
// x 1 54.9, 64 x 8 x 2 57.6; 4096 x 11008 256 x 6 x 2 50.8, 1024 x 2 x 4 71.6; 8192 x 8192 256 x 4 x 4 77.1, x 2 81.0,
// 512 x 2 x 4 81.4, 1024 x 2 x 2 108; 8192 x 22016 512 x 6 x 2 215, x 1 236, x 4 251, 256 x 11 x 1 235.  Non-temporal reads and writes of whole
// lines: 8192 x 8192 77.1 -> 68.5, 8192 x 22016 215 -> 202, 4096 x 11008 and 12288 x 4096 within 2 us; not in a cache 63.5 -> 60.2, 61.8 -> 59.6.
// Binary16 of up to 12288 columns, with digits that four rows share, held to 128 registers (whole calibrations of 600 tokens, 256 x 6 x 2 -> 512 x 3 x 4:
// 4096 x 11008 84.8 -> 83.9, 1000 x 10000 40.1 -> 38.6, 8192 x 12000 185 -> 182.5; with 130 registers 4096 x 11008 93.0; one register is spilled there, in
// binary32 many).  Up to 1024 columns a wavefront to a row, to two rows of more than 2048, which share what they read of a column (whole calibrations, one
// row -> two: 64 tokens 22016 x 256 45.5 -> 39.0, 512 tokens 11008 x 512 33.9 -> 31.4, 2048 tokens 11008 x 1024 44.9 -> 42.1, binary32 2048 tokens 4096 x 768
// 31.2 -> 30.3; 2052 rows within 2 % either way, 6000 tokens 2048 x 1024 28.8 -> 29.5; four rows 600 tokens 22016 x 512 44.5 -> 43.0, binary32 22016 x 1024
// 79.9 -> 82.6).
template <bool F16, bool LINES>
static void launch_rows_for(PassArgs& a, hipStream_t st)
{
    constexpr int64_t kShortK = kWave * 2 * 8;   // columns that a wavefront's two units a lane hold
    static_assert(kCopiesK <= kShortK, "only a wavefront of short rows adds copies up");
    int64_t N = 0;
    for (int i = 0; i < a.n; ++i) N += a.m[i].N;
    if (a.K <= kShortK && N <= 2048) launch_rows<F16, LINES, 64, 2, 1>(a, st);
    else if (a.K <= kShortK) launch_rows<F16, LINES, 64, 2, 2>(a, st);
    else if (a.K <= 4096) launch_rows<F16, LINES, 256, 2, 4>(a, st);
    else if (a.K <= 8192) launch_rows<F16, LINES, 256, 4, F16 ? 4 : 2>(a, st);
    else if (a.K <= 12288) {
        if constexpr (F16) launch_rows<F16, LINES, 512, 3, 4>(a, st);
        else launch_rows<F16, LINES, 256, 6, 2>(a, st);
    }
    else launch_rows<F16, LINES, 512, 6, 2>(a, st);
}

template <bool F16, bool LINES, int BITS, int LEVELS>
static void launch_groups(PassArgs& a, hipStream_t st)
{
    if (a.K <= 1024) weight_pass_groups<F16, LINES, BITS, LEVELS, 64><<<place_blocks(a, kPassRows, 64), 64, 0, st>>>(a);
    else weight_pass_groups<F16, LINES, BITS, LEVELS, 256><<<place_blocks(a, kPassRows, 256), 256, 0, st>>>(a);
}

template <bool F16, bool LINES, int BITS>
static void launch_groups_for(PassArgs& a, int group, hipStream_t st)
{
    switch (group) {
    case 32: return launch_groups<F16, LINES, BITS, 2>(a, st);
    case 64: return launch_groups<F16, LINES, BITS, 3>(a, st);
    case 128: return launch_groups<F16, LINES, BITS, 4>(a, st);
    case 256: return launch_groups<F16, LINES, BITS, 5>(a, st);
    default: return launch_groups<F16, LINES, BITS, 6>(a, st);
    }
}

int launch_weight_pass(PassArgs& a, aweq_dtype dt, int bits, int group, hipStream_t st)
{
    bool lines = dt == AWEQ_F16;
    for (int i = 0; i < a.n; ++i)
        lines = lines && reinterpret_cast<uintptr_t>(a.m[i].W) % 128 == 0 && reinterpret_cast<uintptr_t>(a.m[i].W_hat) % 128 == 0 &&
                (a.m[i].ldw * 2) % 128 == 0 && (a.m[i].ldwh * 2) % 128 == 0;
#define AWEQ_WP(F, L) do { if (bits == 8) launch_rows_for<F, L>(a, st); else if (bits == 4) launch_groups_for<F, L, 4>(a, group, st); else launch_groups_for<F, L, 3>(a, group, st); } while (0)
    if (lines) AWEQ_WP(true, true);
    else if (dt == AWEQ_F16) AWEQ_WP(true, false);
    else AWEQ_WP(false, false);
#undef AWEQ_WP
    return launch_status();
}

int launch_finish(const FinishArgs& fin, int64_t K, hipStream_t st)
{
    calib_finish<<<(unsigned)cdiv(K, kFinishThreads), kFinishThreads, 0, st>>>(fin, K);
    return launch_status();
}

}  // namespace aweq
