// The whole calibration of a layer, or of layers that read the same activation, as one call (Sec. 3: statistics, equalization,
// quantizers, forward, bias correction): what the stage entry points give one after the other, in fewer and larger launches.
//
// A calibration is a chain of passes over X and W with reductions over the whole matrix between them, and every launch of the chain
// costs 4 - 5 us however little it does.  Here the chain is
//   1. column statistics of X and of every W, in one launch (their blocks share the compute units and the pipeline drains once);
//   2. merge of the partial rows, ranges, Eq. 10's scales and the pieces of the ranges over all channels, in one launch;
//   3. int8 path: the activation quantizer, whose blocks find Step and Z from the pieces and add their sums up;
//   4. one pass over every weight: fold, quantise, correct the bias (weight_pass.hip); blocks beside it finish R and p;
//   5. forward: the GEMMs, without column sums (the pass has them); in one launch where several layers have one width.
// Calls that the pass does not take (one scale for the tensor, groups or widths it has no form for) run stages 2b - 5 as they are
// behind 1 and 2; buffers that overlap, or a workspace of the stages' own size, take the stages one by one.
#include "col_stats.hpp"
#include "gemm_i8.hpp"
#include "quant_act.hpp"
#include "weight_pass.hpp"

namespace aweq {

// ---- 1: column statistics of several matrices of K columns
constexpr int kSources = 1 + kMaxMembers;
struct StatsSource {
    const void* M;
    int64_t rows, ld;
    int first_slice, keep;
};
struct StatsSources {
    StatsSource src[kSources];   // X first
    int n;
    int64_t K, rows_per_slice;
    float *pmin, *pmax;          // [slices][K]
    double* psum;
};

template <bool F16>
__global__ __launch_bounds__(kStatsBlock) void calib_stats(StatsSources a)
{
    __shared__ StatsLds<SliceStats<F16>::kCols> s;
    int i = 0;
    while (i + 1 < a.n && (int)blockIdx.y >= a.src[i + 1].first_slice) ++i;
    const StatsSource& m = a.src[i];
    const int64_t r0 = (int64_t)((int)blockIdx.y - m.first_slice) * a.rows_per_slice, o = (int64_t)blockIdx.y * a.K;
    stats_slice<F16>(s, m.M, a.K, m.ld, blockIdx.x, r0, min(m.rows, r0 + a.rows_per_slice), m.keep != 0, a.pmin + o, a.pmax + o, a.psum + o);
}

struct CalibPlan {
    int chunks, x_slices, slices;
    int64_t rows_per_slice;
    int first[kSources];
};

// Slices of equal height over all matrices, all resident at a time: 4 blocks of binary16 to a compute unit (us of the whole calibration, 5 -> 4:
// 14331 x 11008 181.5 -> 178, 65536 x 4096 INT4 150 -> 146, 32768 x 4096 144 -> 127 with the rule of spread_rows), 5 of binary32.
static CalibPlan calib_plan(const int64_t* rows, int n, int64_t K, bool f16)
{
    CalibPlan p;
    p.chunks = (int)cdiv(K, (int64_t)kWave * (f16 ? 8 : 4));
    int64_t total = 0;
    for (int i = 0; i < n; ++i) total += rows[i];
    const int64_t step = kStatsWaves * kRowBatch, most = (f16 ? 1024 : 1280) / p.chunks > n ? (f16 ? 1024 : 1280) / p.chunks : n;
    p.rows_per_slice = cdiv(cdiv(total, most), step) * step;
    for (;;) {
        int64_t slices = 0;
        for (int i = 0; i < n; ++i) { p.first[i] = (int)slices; slices += cdiv(rows[i], p.rows_per_slice); }
        p.slices = (int)slices;
        p.x_slices = n > 1 ? p.first[1] : p.slices;
        if (slices <= most && p.rows_per_slice == spread_rows(p.rows_per_slice)) return p;
        p.rows_per_slice += step;
    }
}

// ---- 2: a block owns 32 columns; its 32 groups of 32 threads take every 32nd partial row each (bound by the latency of these few
// loads) and meet in LDS in a fixed order, so that the fp64 sums are reproducible
constexpr int kMergeCols = kRangeCols, kMergeParts = 32;
struct MergeArgs {
    const float *pmin, *pmax;
    const double* psum;
    int x_slices, slices;
    int64_t K;
    uint64_t T, N;        // rows of X, of all weights
    int enable_awe;
    float *xmin, *xmax, *r_x, *wmin, *wmax, *r_w, *s, *inv_s, *mu_xhat;
    double* xsum;
    uint64_t *count, *wcount;
    float* ext;           // [6][gridDim.x]
    int32_t *colsum, *rowsum;   // nullable: zero for the launch that adds to them, [copies][K] and [T]
    int copies;
    uint32_t* status;
};

__global__ __launch_bounds__(kMergeCols * kMergeParts) void calib_merge(MergeArgs a)
{
    __shared__ float s_f[4][kMergeParts][kMergeCols];
    __shared__ double s_d[2][kMergeParts][kMergeCols];
    const int c = threadIdx.x & (kMergeCols - 1), part = threadIdx.x / kMergeCols;
    const int64_t k = (int64_t)blockIdx.x * kMergeCols + c;
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        if (a.count) *a.count = a.T;
        if (a.wcount) *a.wcount = a.N;
    }
    if (a.colsum && part < a.copies && k < a.K) a.colsum[part * a.K + k] = 0;
    if (a.rowsum)
        for (uint64_t t = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; t < a.T; t += (uint64_t)gridDim.x * blockDim.x) a.rowsum[t] = 0;
    float lo = INFINITY, hi = -INFINITY, wlo = INFINITY, whi = -INFINITY;
    double sum = 0.0, wsum = 0.0;
    if (k < a.K) {
        for (int j = part; j < a.x_slices; j += kMergeParts) {
            lo = fminf(lo, a.pmin[(int64_t)j * a.K + k]);
            hi = fmaxf(hi, a.pmax[(int64_t)j * a.K + k]);
            sum += a.psum[(int64_t)j * a.K + k];
        }
        for (int j = a.x_slices + part; j < a.slices; j += kMergeParts) {
            wlo = fminf(wlo, a.pmin[(int64_t)j * a.K + k]);
            whi = fmaxf(whi, a.pmax[(int64_t)j * a.K + k]);
            wsum += a.psum[(int64_t)j * a.K + k];
        }
    }
    s_f[0][part][c] = lo; s_f[1][part][c] = hi; s_f[2][part][c] = wlo; s_f[3][part][c] = whi;
    s_d[0][part][c] = sum; s_d[1][part][c] = wsum;
    __syncthreads();
    // one quantity a group of 32 threads, left in its row 0
    if (part < 4) {
        float v = s_f[part][0][c];
#pragma unroll
        for (int q = 1; q < kMergeParts; ++q) v = part & 1 ? fmaxf(v, s_f[part][q][c]) : fminf(v, s_f[part][q][c]);
        s_f[part][0][c] = v;
    } else if (part < 6) {
        double v = s_d[part - 4][0][c];
#pragma unroll
        for (int q = 1; q < kMergeParts; ++q) v += s_d[part - 4][q][c];
        s_d[part - 4][0][c] = v;
    }
    __syncthreads();
    if (part != 0) return;
    uint32_t st = 0;
    float hlo = INFINITY, hhi = -INFINITY;
    if (k < a.K) {
        lo = s_f[0][0][c]; hi = s_f[1][0][c]; wlo = s_f[2][0][c]; whi = s_f[3][0][c];
        sum = s_d[0][0][c]; wsum = s_d[1][0][c];
        // a non-finite input makes the fp64 sum (Inf / NaN) or an extreme (Inf) non-finite
        if (!isfinite(sum) || isinf(lo) || isinf(hi) || !isfinite(wsum) || isinf(wlo) || isinf(whi)) st |= AWEQ_ST_NONFINITE;
        a.xmin[k] = lo; a.xmax[k] = hi; a.xsum[k] = sum; a.r_x[k] = hi - lo;
        a.wmin[k] = wlo; a.wmax[k] = whi; a.r_w[k] = whi - wlo;
        const float sk = channel_scale(lo, hi, wlo, whi, a.enable_awe, st), is = 1.0f / sk;
        a.s[k] = sk;
        a.inv_s[k] = is;
        a.mu_xhat[k] = (float)((sum / (double)a.T) * (double)is);
        // (a correctly rounded multiply by a positive constant is monotone: the scaled extremes are the extremes of the scaled column)
        hlo = lo * is;
        hhi = hi * is;
    } else {
        lo = INFINITY; hi = -INFINITY; wlo = INFINITY; whi = -INFINITY;
    }
    raise_status(a.status, st);
    const float e[6] = {group_allreduce<5>(lo, OpMin()), group_allreduce<5>(hi, OpMax()), group_allreduce<5>(wlo, OpMin()),
                        group_allreduce<5>(whi, OpMax()), group_allreduce<5>(hlo, OpMin()), group_allreduce<5>(hhi, OpMax())};
    if (c == 0) {
#pragma unroll
        for (int i = 0; i < 6; ++i) a.ext[i * gridDim.x + blockIdx.x] = e[i];
    }
}

// ---- workspace: what later launches read (the pieces of the ranges; the code sums), then partial rows (of the statistics; of the
// stages' quantizer)
static size_t ext_bytes(int64_t K) { return (size_t)cdiv(6 * cdiv(K, kRangeCols) * 4, 256) * 256; }
static size_t sum_bytes(int64_t K, int copies) { return (size_t)cdiv(K * 4 * copies, 256) * 256; }
static size_t kept_bytes(int64_t K, int copies) { return ext_bytes(K) + sum_bytes(K, copies); }
static size_t partial_bytes(const CalibPlan& p, int64_t K) { return (size_t)p.slices * (size_t)K * 16; }

// for any division of N rows over up to kMaxMembers weights: a plan has at most max(1280 / chunks, n) slices
static size_t calibrate_ws_bytes(int64_t T, int64_t K, int64_t N, int copies)
{
    if (N <= 0) return 0;
    size_t most = 0;
    for (const bool f16 : {false, true}) {
        const int64_t chunks = cdiv(K, (int64_t)kWave * (f16 ? 8 : 4));
        const int64_t rows = cdiv(T, kStatsWaves * kRowBatch) + cdiv(N, kStatsWaves * kRowBatch) + kMaxMembers - 1;
        int64_t slices = 1280 / chunks > kSources ? 1280 / chunks : kSources;
        if (slices > rows) slices = rows;
        const size_t b = (size_t)slices * (size_t)K * 16;
        if (b > most) most = b;
    }
    const size_t qa = quant_act_ws_bytes(T, K);
    return kept_bytes(K, copies) + (most > qa ? most : qa);
}
size_t calibrate_ws_bytes(int64_t T, int64_t K, int64_t N) { return calibrate_ws_bytes(T, K, N, sum_copies(K)); }

// one copy of the code sums for few tokens, and in a workspace with no room for more
static int copies_in(const aweq_calib_layer& l, const aweq_calib_weight* w, int n)
{
    int64_t N = 0;
    for (int i = 0; i < n; ++i) N += w[i].N;
    return l.T > copies_tokens(l.K) && l.ws_bytes >= calibrate_ws_bytes(l.T, l.K, N) ? sum_copies(l.K) : 1;
}

// no buffer that is written shares a byte with another buffer
static bool buffers_apart(const aweq_calib_layer& l, const aweq_calib_weight* w, int n)
{
    struct Item { uintptr_t b, e; bool out; } it[40 + 16 * kMaxMembers];
    int m = 0;
    auto add = [&](const Span& s, bool out) {
        if (s.p && s.bytes > 0) it[m++] = {reinterpret_cast<uintptr_t>(s.p), reinterpret_cast<uintptr_t>(s.p) + (uintptr_t)s.bytes, out};
    };
    const int64_t K = l.K, T = l.T;
    add(matrix_span(l.X, T, K, l.ldx, dtype_size(l.dt)), false);
    for (const float* v : {l.xmin, l.xmax, l.r_x, l.p_x, l.wmin, l.wmax, l.r_w, l.p_w, l.s, l.inv_s, l.mu_xhat}) add({v, K * 4}, true);
    add({l.xsum, K * 8}, true);
    for (const void* v : {(const void*)l.count, (const void*)l.wcount, (const void*)l.xhat_range}) add({v, 8}, true);
    for (const void* v : {(const void*)l.R_x, (const void*)l.R_w, (const void*)l.act_step, (const void*)l.act_zero, (const void*)l.status}) add({v, 4}, true);
    add({l.xq, T * panel_count(K) * kPanel}, true);
    add({l.rowsum_x, T * 4}, true);
    add({l.colsum_xq, K * 8}, true);
    add({l.ws, (int64_t)l.ws_bytes}, true);
    for (int i = 0; i < n; ++i) {
        const aweq_calib_weight& v = w[i];
        // (a folded weight in the place of its weight is as good: a block has read the rows that it writes)
        if (v.W != v.W_hat || v.ldw != v.ldwh) add(matrix_span(v.W, v.N, K, v.ldw, dtype_size(l.dt)), false);
        add(matrix_span(v.W_hat, v.N, K, v.ldwh, dtype_size(l.dt)), true);
        const int64_t slices = l.group > 0 ? v.N * (K / l.group) : l.group == 0 ? v.N : 1;
        add({v.codes, l.bits == 8 && l.group <= 0 ? v.N * panel_count(K) * kPanel : v.N * (K / 8) * l.bits}, true);
        add({v.step_w, slices * 4}, true);
        add({v.zero_w, slices * 4}, true);
        add({v.bias_in, v.N * 4}, false);
        for (const void* q : {(const void*)v.rowsum_w, (const void*)v.delta, (const void*)v.bias_out}) add({q, v.N * 4}, true);
        add({v.colsum_acc, v.N * 8}, true);
        add(matrix_span(v.out_i32, T, v.N, v.N, 4), true);
        add(matrix_span(v.out_deq, T, v.N, v.N, dtype_size(l.dt)), true);
    }
    for (int i = 1; i < m; ++i) {   // by address
        const Item x = it[i];
        int j = i;
        for (; j > 0 && it[j - 1].b > x.b; --j) it[j] = it[j - 1];
        it[j] = x;
    }
    uintptr_t end = 0, end_out = 0;
    for (int i = 0; i < m; ++i) {
        if (it[i].b < (it[i].out ? end : end_out)) return false;
        if (it[i].e > end) end = it[i].e;
        if (it[i].out && it[i].e > end_out) end_out = it[i].e;
    }
    return true;
}

// launches 1 and 2 take the call: everything they need is there, aligned, in reach and apart
static bool fused_front(const aweq_calib_layer& l, const aweq_calib_weight* w, int n)
{
    if (n < 1 || n > kMaxMembers || !l.X || !l.ws || (l.dt != AWEQ_F16 && l.dt != AWEQ_F32)) return false;
    for (const void* p : {(const void*)l.xmin, (const void*)l.xmax, (const void*)l.xsum, (const void*)l.r_x, (const void*)l.R_x, (const void*)l.wmin,
                          (const void*)l.wmax, (const void*)l.r_w, (const void*)l.R_w, (const void*)l.s, (const void*)l.inv_s,
                          (const void*)l.xhat_range, (const void*)l.mu_xhat, (const void*)l.act_step, (const void*)l.act_zero})
        if (!p) return false;
    if (l.T <= 0 || l.K <= 0 || (l.K % 8) != 0 || l.K > (1 << 26) || l.ldx < l.K) return false;
    if (l.enable_awe < 0 || l.enable_awe > AWEQ_SCALE_ABSMAX || (l.bits != 8 && l.bits != 4 && l.bits != 3)) return false;
    const size_t e = dtype_size(l.dt);
    if (!aligned16(l.X) || (l.ldx * e) % 16 != 0 || !aligned16(l.ws) || !aligned16(l.s) || !aligned16(l.mu_xhat)) return false;
    int64_t N = 0;
    for (int i = 0; i < n; ++i) {
        const aweq_calib_weight& v = w[i];
        if (!v.W || !v.W_hat || !v.codes || !v.step_w || !v.zero_w || !v.delta || !v.bias_out) return false;
        if (v.N <= 0 || v.N > 0x7fffffffll || v.ldw < l.K || v.ldwh < l.K) return false;
        if (!aligned16(v.W) || !aligned16(v.W_hat) || (v.ldw * e) % 16 != 0 || (v.ldwh * e) % 16 != 0 || !aligned16(v.codes)) return false;
        N += v.N;
    }
    if (l.w8a8 && (!l.colsum_xq || (l.forward && (!l.xq || !l.rowsum_x || !aligned16(l.xq) || l.K > 32768)))) return false;
    return l.ws_bytes >= calibrate_ws_bytes(l.T, l.K, N, 1) && buffers_apart(l, w, n);
}

// pass: the quantizer adds its sums up, to what the merge zeroes
static int run_front(const aweq_calib_layer& l, const aweq_calib_weight* w, int n, bool pass, FinishArgs& fin, hipStream_t st)
{
    int64_t rows[kSources] = {l.T}, N = 0;
    for (int i = 0; i < n; ++i) { rows[1 + i] = w[i].N; N += w[i].N; }
    const bool f16 = l.dt == AWEQ_F16;
    const int copies = copies_in(l, w, n);
    const CalibPlan p = calib_plan(rows, n + 1, l.K, f16);
    if (p.slices > 65535) return AWEQ_ERR_SHAPE;
    StatsSources a;
    a.n = n + 1; a.K = l.K; a.rows_per_slice = p.rows_per_slice;
    a.psum = reinterpret_cast<double*>(reinterpret_cast<char*>(l.ws) + kept_bytes(l.K, copies));
    a.pmin = reinterpret_cast<float*>(a.psum + (size_t)p.slices * l.K);
    a.pmax = a.pmin + (size_t)p.slices * l.K;
    for (int i = 0; i <= n; ++i) {
        StatsSource& s = a.src[i];
        s.M = i ? w[i - 1].W : l.X;
        s.ld = i ? w[i - 1].ldw : l.ldx;
        s.rows = rows[i];
        s.first_slice = p.first[i];
        s.keep = rows[i] * l.K * (int64_t)dtype_size(l.dt) <= kKeepBytes;   // (the rule of aweq_calib_stats)
    }
    const dim3 grid((unsigned)p.chunks, (unsigned)p.slices);
    if (f16) calib_stats<true><<<grid, kStatsBlock, 0, st>>>(a);
    else calib_stats<false><<<grid, kStatsBlock, 0, st>>>(a);
    const unsigned blocks = (unsigned)cdiv(l.K, kMergeCols);
    const MergeArgs m = {a.pmin, a.pmax, a.psum, p.x_slices, p.slices, l.K, (uint64_t)l.T, (uint64_t)N, l.enable_awe, l.xmin, l.xmax, l.r_x,
                         l.wmin, l.wmax, l.r_w, l.s, l.inv_s, l.mu_xhat, l.xsum, l.count, l.wcount, reinterpret_cast<float*>(l.ws),
                         pass && l.w8a8 ? reinterpret_cast<int32_t*>(reinterpret_cast<char*>(l.ws) + ext_bytes(l.K)) : nullptr,
                         pass && l.w8a8 && l.forward && quant_act_adds_rows(l.K) ? l.rowsum_x : nullptr, copies, l.status};
    calib_merge<<<blocks, kMergeCols * kMergeParts, 0, st>>>(m);
    fin = {{m.ext, (int)blocks, l.xhat_range, l.act_step, l.act_zero}, l.r_x, l.r_w, l.R_x, l.R_w, l.p_x, l.p_w, nullptr, nullptr, l.status};
    return launch_status();
}

// The forward of layers of one width with binary16 outputs in one launch.  false: nothing was launched.
static bool group_forward(const aweq_calib_layer& l, const aweq_calib_weight* w, int n, hipStream_t st)
{
    static_assert(kMaxMembers <= kGroupMost, "every weight has its operands");
    if (n < 2 || l.dt != AWEQ_F16 || (w[0].N % 4) != 0) return false;
    GroupArgs g = {};
    g.A = l.xq; g.T = l.T; g.N = w[0].N; g.K = l.K; g.out_f16 = 1; g.ldo = w[0].N;
    g.act_step = l.act_step; g.act_zero = l.act_zero; g.rowsum_x = l.rowsum_x; g.status = l.status;
    for (int i = 0; i < n; ++i) {
        const aweq_calib_weight& v = w[i];
        if (v.N != g.N || v.out_i32 || !v.out_deq || !aligned16(v.out_deq) || !aligned16(v.step_w) || !aligned16(v.zero_w) || !aligned16(v.rowsum_w) ||
            (v.bias_in && !aligned16(v.bias_in)))
            return false;
        g.m[i] = {reinterpret_cast<const int8_t*>(v.codes), v.out_deq, v.step_w, v.zero_w, v.rowsum_w, v.bias_in};
    }
    return launch_gemm_i8_group(g, n, st) == AWEQ_OK;
}

static int run_calibration(const aweq_calib_layer& l, const aweq_calib_weight* w, int n, void* stream)
{
    hipStream_t st = as_stream(stream);
    const bool front = fused_front(l, w, n);
    bool pass = front;
    for (int i = 0; pass && i < n; ++i) pass = weight_pass_takes(l.bits, l.group, l.w8a8 != 0, w[i].N, l.K, (uint64_t)l.T);
    // fold and quantise in calls of their own: aweq_fold_quant_weight has one scale per output channel only
    const bool fold = l.group != 0 || (n == 1 && !l.fused_weight_pass);
    int rc;
    FinishArgs fin;
    if (front) {
        rc = run_front(l, w, n, pass, fin, st);
        if (rc != AWEQ_OK) return rc;
    }
    if (pass) {
        char* const ws = reinterpret_cast<char*>(l.ws);
        int32_t* const colsum = reinterpret_cast<int32_t*>(ws + ext_bytes(l.K));
        const int copies = copies_in(l, w, n);
        if (l.w8a8) {
            rc = launch_quant_act(l.X, l.dt, l.T, l.K, l.ldx, l.inv_s, l.act_step, l.act_zero, l.forward ? l.xq : nullptr,
                                  l.forward ? l.rowsum_x : nullptr, nullptr, nullptr, l.status, st, &fin.range, colsum, copies);
            if (rc != AWEQ_OK) return rc;
            fin.range.act_step = nullptr;   // (the quantizer has written it)
            fin.colsum = colsum;
            fin.colsum_xq = reinterpret_cast<long long*>(l.colsum_xq);
        }
        PassArgs a;
        a.n = n; a.K = l.K; a.s = l.s; a.mu = l.mu_xhat; a.count = (uint64_t)l.T; a.colsum = colsum; a.copies = copies;
        a.act_step = l.act_step; a.act_zero = l.act_zero; a.enable_bc = l.enable_bc; a.status = l.status; a.fin = fin;
        for (int i = 0; i < n; ++i)
            a.m[i] = {w[i].W, w[i].W_hat, reinterpret_cast<uint8_t*>(w[i].codes), w[i].step_w, w[i].zero_w, w[i].rowsum_w, w[i].bias_in, w[i].delta,
                      w[i].bias_out, l.forward ? reinterpret_cast<long long*>(w[i].colsum_acc) : nullptr, w[i].N, w[i].ldw, w[i].ldwh, 0u};
        rc = launch_weight_pass(a, l.dt, l.bits, l.group, st);
        if (rc != AWEQ_OK) return rc;
        if (l.w8a8 && l.forward && group_forward(l, w, n, st)) return launch_status();
        for (int i = 0; l.w8a8 && l.forward && i < n; ++i) {
            if (!w[i].out_i32 && !w[i].out_deq) continue;
            rc = aweq_w8a8_gemm(l.xq, AWEQ_I8, l.T, l.K, l.K, nullptr, l.act_step, l.act_zero, nullptr, l.rowsum_x, nullptr,
                                reinterpret_cast<const int8_t*>(w[i].codes), w[i].N, w[i].step_w, w[i].zero_w, 0, w[i].rowsum_w, w[i].bias_in,
                                w[i].out_i32, w[i].out_deq, l.dt, w[i].N, nullptr, nullptr, 0, l.status, stream);
            if (rc != AWEQ_OK) return rc;
        }
        return AWEQ_OK;
    }

    // the stages one by one
    if (front) {
        rc = launch_finish(fin, l.K, st);
        if (rc != AWEQ_OK) return rc;
        for (int i = 0; fold && i < n; ++i) launch_fold(w[i].W, w[i].W_hat, l.dt, w[i].N, l.K, w[i].ldw, w[i].ldwh, l.s, st);
    } else {
        rc = aweq_calib_stats(l.X, l.dt, l.T, l.K, l.ldx, l.xmin, l.xmax, l.xsum, l.count, 0, 1, l.r_x, l.R_x, l.p_x, l.ws, l.ws_bytes, l.status, stream);
        for (int i = 0; rc == AWEQ_OK && i < n; ++i)   // (min of mins, max of maxes over the weights)
            rc = aweq_calib_stats(w[i].W, l.dt, w[i].N, l.K, w[i].ldw, l.wmin, l.wmax, nullptr, l.wcount, i > 0, i == n - 1, l.r_w, l.R_w, l.p_w, l.ws,
                                  l.ws_bytes, l.status, stream);
        if (rc != AWEQ_OK) return rc;
        rc = aweq_equalize(l.xmin, l.xmax, l.xsum, (uint64_t)l.T, l.wmin, l.wmax, l.K, l.enable_awe, l.s, l.inv_s, fold ? w[0].W : nullptr,
                           fold ? w[0].W_hat : nullptr, l.dt, w[0].N, w[0].ldw, w[0].ldwh, nullptr, l.xhat_range, l.mu_xhat, l.act_step, l.act_zero,
                           l.status, stream);
        for (int i = 1; rc == AWEQ_OK && fold && i < n; ++i) {
            rc = check_fold_args(w[i].W, w[i].W_hat, l.dt, w[i].N, l.K, w[i].ldw, w[i].ldwh);
            if (rc == AWEQ_OK) launch_fold(w[i].W, w[i].W_hat, l.dt, w[i].N, l.K, w[i].ldw, w[i].ldwh, l.s, st);
        }
        if (rc != AWEQ_OK) return rc;
    }
    for (int i = 0; i < n; ++i) {
        int32_t* const rowsum = l.bits == 8 && l.group <= 0 ? w[i].rowsum_w : nullptr;
        rc = fold ? aweq_quant_weight(w[i].W_hat, l.dt, w[i].N, l.K, w[i].ldwh, l.bits, l.group, w[i].codes, w[i].step_w, w[i].zero_w, rowsum, l.ws,
                                      l.ws_bytes, l.status, stream)
                  : aweq_fold_quant_weight(w[i].W, l.dt, w[i].N, l.K, w[i].ldw, l.s, w[i].W_hat, w[i].ldwh, l.bits, w[i].codes, w[i].step_w,
                                           w[i].zero_w, rowsum, l.status, stream);
        if (rc != AWEQ_OK) return rc;
    }
    const int wg = l.group < 0 ? -1 : 0;   // per-tensor weights (Sec. 3): one (Step, Z), read as such by stages 4 and 5
    if (!l.w8a8) {
        for (int i = 0; i < n; ++i) {
            rc = aweq_bias_correct(AWEQ_BIAS_WEIGHT_ONLY, w[i].W_hat, l.dt, w[i].N, l.K, w[i].ldwh, l.mu_xhat, (uint64_t)l.T, nullptr, nullptr, nullptr,
                                   nullptr, nullptr, w[i].codes, l.bits, l.group, w[i].step_w, w[i].zero_w, w[i].bias_in, w[i].delta, w[i].bias_out,
                                   l.enable_bc, l.status, stream);
            if (rc != AWEQ_OK) return rc;
        }
        return AWEQ_OK;
    }
    if (!l.forward || n > 1) {   // (several layers: the codes of X once)
        rc = aweq_quant_act(l.X, l.dt, l.T, l.K, l.ldx, l.inv_s, l.act_step, l.act_zero, l.forward ? l.xq : nullptr, l.forward ? l.rowsum_x : nullptr,
                            l.colsum_xq, l.ws, l.ws_bytes, l.status, stream);
        if (rc != AWEQ_OK) return rc;
    }
    for (int i = 0; i < n; ++i) {
        const int8_t* const codes = reinterpret_cast<const int8_t*>(w[i].codes);
        if (l.forward) {
            rc = n > 1 ? aweq_w8a8_gemm(l.xq, AWEQ_I8, l.T, l.K, l.K, nullptr, l.act_step, l.act_zero, nullptr, l.rowsum_x, nullptr, codes, w[i].N,
                                        w[i].step_w, w[i].zero_w, wg, w[i].rowsum_w, w[i].bias_in, w[i].out_i32, w[i].out_deq, l.dt, w[i].N,
                                        w[i].colsum_acc, nullptr, 0, l.status, stream)
                       : aweq_w8a8_gemm(l.X, l.dt, l.T, l.K, l.ldx, l.inv_s, l.act_step, l.act_zero, l.xq, l.rowsum_x, l.colsum_xq, codes, w[i].N,
                                        w[i].step_w, w[i].zero_w, wg, w[i].rowsum_w, w[i].bias_in, w[i].out_i32, w[i].out_deq, l.dt, w[i].N,
                                        w[i].colsum_acc, l.ws, l.ws_bytes, l.status, stream);
            if (rc != AWEQ_OK) return rc;
        }
        rc = aweq_bias_correct(AWEQ_BIAS_W8A8, w[i].W_hat, l.dt, w[i].N, l.K, w[i].ldwh, l.mu_xhat, (uint64_t)l.T, l.forward ? w[i].colsum_acc : nullptr,
                               l.colsum_xq, w[i].rowsum_w, l.act_step, l.act_zero, l.forward ? nullptr : w[i].codes, 8, wg, w[i].step_w, w[i].zero_w,
                               w[i].bias_in, w[i].delta, w[i].bias_out, l.enable_bc, l.status, stream);
        if (rc != AWEQ_OK) return rc;
    }
    return AWEQ_OK;
}

}  // namespace aweq

extern "C" int aweq_calibrate(const aweq_calib_layer* layer, const aweq_calib_weight* weights, int n_weights, void* stream)
{
    if (!layer || !weights) return AWEQ_ERR_NULL;
    if (n_weights < 1) return AWEQ_ERR_SHAPE;
    // the int8 path multiplies 8-bit codes in K-panels, with one scale per output channel or per tensor
    if (layer->w8a8 && layer->bits != 8) return AWEQ_ERR_BITS;
    if (layer->w8a8 && layer->group != 0 && layer->group != -1) return AWEQ_ERR_GROUP;
    // what the int8 path's bias correction reads, whichever route the call takes
    for (int i = 0; layer->w8a8 && i < n_weights; ++i)
        if (!weights[i].rowsum_w || (layer->forward && !weights[i].colsum_acc)) return AWEQ_ERR_NULL;
    return aweq::run_calibration(*layer, weights, n_weights, stream);
}
