// Stage 4b for few tokens (decoding, small batches): the int8 GEMM when one read of the weight codes is nearly all
// there is to do.
//
// A workgroup of 8 wavefronts owns 16 NT output channels x 16 TT tokens and splits K between its wavefronts, whose
// int32 partial sums meet in LDS, so that one token spreads over N / 16 workgroups instead of N / 256.  Both
// operands come straight from their K-panels (16 rows of a panel are 1 KiB contiguous) in the operand order of
// v_mfma_i32_16x16x64_i8: lane l holds row l % 16, bytes 16 (l / 16) .. + 15 of the panel row.
//
// Bound by the read of the weight.  Measured (us per call on the device, codes given, binary16 output, the same weight every call; before =
// 256 x 256 tiles; from 128 tokens on also the kernel for some hundred tokens, where it is modelled to take less):
//   tokens          1             32            64            128           256
//   4096 x 4096     37.7 ->  3.8  38.4 ->  5.2  38.9 ->  6.2  40.8 ->  8.0  43.0 -> 10.6
//   8192 x 8192     68.3 -> 12.4  68.5 -> 13.4  69.3 -> 14.2  71.4 -> 18.2  72.7 -> 28.9
//   22016 x 8192    71.8 -> 30.6  70.4 -> 31.1  71.3 -> 31.7  73.2 -> 40.6    80 -> 50.2
// (22016 x 8192 at one token: 180 MB, 5.9 TB/s.)
#include "act_unit.hpp"
#include "gemm_i8.hpp"

namespace aweq {
namespace few {

typedef int v4i __attribute__((ext_vector_type(4)));

constexpr int kThreads = 512;
constexpr int kWaves = kThreads / kWave;

// QX: 0: the tokens' codes are in memory (g.A).  1 / 2: every workgroup quantises the few binary16 / binary32 tokens (QuantIn) for
// itself while its first weights are on their way, the first workgroup also for the caller: a second launch costs more
// than the repeated work.  TQ: their number, 4 for three too.  Loads return in order, so the tokens, their scales and the epilogue's constants are
// requested ahead of the weights; behind them the quantizer waited for the weights first (us a call, weights in the caches, before -> now, with reads of the tokens that
// leave them in the caches for the other workgroups: one token 4096 x 4096 6.4 -> 5.15, 8192 x 8192 16.0 -> 13.6, 4096 x 16384 18.0 -> 15.6,
// 11008 x 4096 10.85 -> 9.3; four tokens 16384 x 4096 15.1 -> 12.95).
template <int TT, int NT, int D, int QX, int TQ>
__global__ __launch_bounds__(kThreads) void gemm_i8_few(GemmArgs g, QuantIn in)
{
    extern __shared__ __attribute__((aligned(16))) int red[];   // [wave][TT NT][lane][4], then (QX) the tokens' codes, K padded to panels
    __shared__ int s_rs[kQuantTokens];
    const int lane = threadIdx.x & (kWave - 1);
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x / kWave));
    const int r = lane & 15, q = lane >> 4;
    const int64_t n0 = (int64_t)blockIdx.x * (16 * NT), t0 = (int64_t)(g.run + (int)blockIdx.y) * (16 * TT);   // (run: the launch's first token tile)
    const int np = (int)panel_count(g.K);
    const int rows_left = (int)min(g.N - n0, (int64_t)(16 * NT)) - 1, tokens_left = (int)min(g.T - t0, (int64_t)(16 * TT)) - 1;

    // rows past the edge re-read the last valid row; their results are never stored
    uint32_t wo[NT], xo[TT];
#pragma unroll
    for (int j = 0; j < NT; ++j) wo[j] = (uint32_t)min(16 * j + r, rows_left) * kPanel + q * 16;
#pragma unroll
    for (int i = 0; i < TT; ++i) xo[i] = (uint32_t)min(16 * i + r, tokens_left) * kPanel + q * 16;
    const int8_t* const wbase = g.B + n0 * kPanel;
    const int8_t* const xbase = g.A + t0 * kPanel;
    const int64_t wp = g.N * kPanel, xp = g.T * kPanel;

    v4i acc[TT][NT];
#pragma unroll
    for (int i = 0; i < TT; ++i)
#pragma unroll
        for (int j = 0; j < NT; ++j) acc[i][j] = v4i{0, 0, 0, 0};

    // Panels wave, wave + 8, ... go through a ring of D slots, each refilled as soon as it has been multiplied; no load sits in a branch but
    // the last ones.  The depths (at the launch) are the best measured of 1 - 8; more cost wavefronts, and the read of the weight is at the
    // memory's rate between the launch's 2.7 us and its end (us, batches issued once the last one had arrived -> ring, weight in
    // the caches: one token 4096 x 4096 5.15 -> 4.9, 16 tokens 4096 x 11008 15.1 -> 14.2, 8192 x 8192 17.7 -> 16.9, 32 tokens 4096 x 4096
    // 9.0 -> 8.5, 4096 x 11008 16.8 -> 15.6, 64 tokens 8192 x 8192 19.1 -> 18.6; wide layers within 1 %).
    const int cnt = max((np - wave + kWaves - 1) / kWaves, 0);
    v4i w[D][NT], x[D][TT];
    auto load = [&](int d, int i) {
        const int p = wave + i * kWaves;
#pragma unroll
        for (int j = 0; j < NT; ++j) w[d][j] = *reinterpret_cast<const v4i*>(wbase + p * wp + wo[j]);
        if constexpr (QX == 0) {
#pragma unroll
            for (int t = 0; t < TT; ++t) x[d][t] = *reinterpret_cast<const v4i*>(xbase + p * xp + xo[t]);
        }
    };
    // (QX) A thread has every kThreads-th unit of 8 values of each token, at most kRounds of them
    constexpr int kRounds = TQ == 1 ? 4 : 2;
    static_assert(QX == 0 || TQ * kRounds * kThreads * 8 >= kQuantFewBytes, "every code has a thread");
    const int units = (int)(g.K / 8), padded = np * (kPanel / 8);
    RawUnit<QX == 1> raw[QX != 0 ? kRounds : 1][QX != 0 ? TQ : 1];
    Float4 is[QX != 0 ? kRounds : 1][2];
    if constexpr (QX != 0) {
#pragma unroll
        for (int i = 0; i < kRounds; ++i) {
            if (i * kThreads >= padded) break;
            const int u = min(i * kThreads + (int)threadIdx.x, units - 1);   // (past K the last unit again, whose codes are not kept)
#pragma unroll
            for (int t = 0; t < TQ; ++t)
                if (TQ <= 2 || t < (int)g.T) raw[i][t].load_shared(in.X, t * in.ldx + u * 8);
            is[i][0] = *reinterpret_cast<const Float4*>(in.inv_s + u * 8);
            is[i][1] = *reinterpret_cast<const Float4*>(in.inv_s + u * 8 + 4);
        }
    }
    // What the epilogue needs of a channel (a token) is requested here by one thread each and waits in LDS: at the end, one round trip after the
    // other, it took 1 - 2 us
    constexpr int kChannels = 16 * NT, kTokens = 16 * TT;
    static_assert(kChannels + kTokens <= kThreads, "a thread each");
    __shared__ double s_scale[kChannels], s_bias[kChannels];
    __shared__ unsigned s_cn[kChannels], s_zw[kChannels], s_rx[kTokens];
    float e_step = 0.0f, e_bias = 0.0f, e_sx = 0.0f;
    int e_zw = 0, e_rw = 0, e_zx = 0;
    const int e_tok = (int)threadIdx.x - kChannels;
    auto request_constants = [&]() {
        if (!g.out_deq) return;
        e_zx = *g.act_zero;
        e_sx = *g.act_step;
        if ((int)threadIdx.x <= rows_left) {
            const int64_t n = n0 + threadIdx.x, pi = g.w_per_tensor ? 0 : n;
            e_step = g.step_w[pi];
            e_zw = g.zero_w[pi];
            e_rw = g.rowsum_w[n];
            if (g.bias) e_bias = g.bias[n];
        } else if (QX == 0 && e_tok >= 0 && e_tok <= tokens_left) {
            e_rw = g.rowsum_x[t0 + e_tok];
        }
    };
    if constexpr (QX != 0) request_constants();   // (with the tokens, ahead of the weights)
    if (cnt >= D) {
#pragma unroll
        for (int d = 0; d < D; ++d) load(d, d);
    } else {
#pragma unroll
        for (int d = 0; d < D; ++d)
            if (d < cnt) load(d, d);
    }
    if constexpr (QX == 0) request_constants();
    int8_t* const codes = reinterpret_cast<int8_t*>(red + kWaves * TT * NT * kWave * 4);
    if constexpr (QX != 0) {
        const ActParams ap = quot_params(*g.act_step, *g.act_zero);
        uint32_t st = 0;
        float big = 0.0f;
        const int T = (int)g.T;
        int rs[TQ];
#pragma unroll
        for (int t = 0; t < TQ; ++t) rs[t] = 0;
        if (threadIdx.x < kQuantTokens) s_rs[threadIdx.x] = 0;
        __syncthreads();
#pragma unroll
        for (int i = 0; i < kRounds; ++i) {
            if (i * kThreads >= padded) break;
            const int u = i * kThreads + (int)threadIdx.x;
            float isf[8];
#pragma unroll
            for (int e = 0; e < 4; ++e) { isf[e] = is[i][0].f[e]; isf[4 + e] = is[i][1].f[e]; }
#pragma unroll
            for (int t = 0; t < TQ; ++t) {
                if (TQ > 2 && t >= T) break;
                float xf[8];
                raw[i][t].get(xf);
                int r8 = 0;
                uint2 c = act_unit_any<QX == 1>(xf, isf, ap, r8, big, st);
                if (u >= units) { c = make_uint2(0u, 0u); r8 = 0; }   // (the zero fill of the last panel)
                rs[t] += r8;
                if (u >= padded) continue;
                *reinterpret_cast<uint2*>(codes + (t * padded + u) * 8) = c;
                if (blockIdx.x == 0) *reinterpret_cast<uint2*>(in.xq + ((int64_t)(u >> 3) * T + t) * kPanel + (u & 7) * 8) = c;
            }
        }
#pragma unroll
        for (int t = 0; t < TQ; ++t) {
            if (TQ > 2 && t >= T) break;
            rs[t] = wave_allreduce(rs[t], OpAdd());
            if (lane == 0) atomicAdd(&s_rs[t], rs[t]);
        }
        if (big >= 16777216.0f) st |= AWEQ_ST_BIGQUOT;
        if (blockIdx.x == 0) raise_status(g.status, st);
        __syncthreads();
        if (blockIdx.x == 0 && in.rowsum_x && (int)threadIdx.x < (int)g.T) in.rowsum_x[threadIdx.x] = s_rs[threadIdx.x];
    }
    const int8_t* const own = codes + min(r, (int)g.T - 1) * np * kPanel + q * 16;   // (QX: one row of 16 tokens)
    auto mul = [&](int d, int i) {
        if constexpr (QX != 0) x[d][0] = *reinterpret_cast<const v4i*>(own + (wave + i * kWaves) * kPanel);
#pragma unroll
        for (int j = 0; j < NT; ++j)
#pragma unroll
            for (int t = 0; t < TT; ++t) acc[t][j] = __builtin_amdgcn_mfma_i32_16x16x64_i8(w[d][j], x[d][t], acc[t][j], 0, 0, 0);
    };
    if (cnt >= D) {
        int i = 0;
        for (; i + 2 * D <= cnt; i += D) {
#pragma unroll
            for (int d = 0; d < D; ++d) { mul(d, i + d); load(d, i + D + d); }
        }
        const int rest = cnt - i - D;   // panels not requested yet, fewer than D
#pragma unroll
        for (int d = 0; d < D; ++d) {
            mul(d, i + d);
            if (d < rest) load(d, i + D + d);
        }
#pragma unroll
        for (int d = 0; d < D - 1; ++d)
            if (d < rest) mul(d, i + D + d);
    } else {
#pragma unroll
        for (int d = 0; d < D - 1; ++d)
            if (d < cnt) mul(d, d);
    }

    // register v of lane l is output channel 4 (l / 16) + v of the 16, token l % 16
    constexpr int kTiles = TT * NT;
#pragma unroll
    for (int i = 0; i < TT; ++i)
#pragma unroll
        for (int j = 0; j < NT; ++j) *reinterpret_cast<v4i*>(red + ((wave * kTiles + i * NT + j) * kWave + lane) * 4) = acc[i][j];
    __shared__ long long s_col[TT][16 * NT];
    uint32_t est = 0;
    if (g.out_deq) {
        // the tiled kernel's arithmetic: the integer part in wrap-around 32 bits, scaled and shifted in fp64
        const int zx = e_zx - 128, zw = e_zw - 128;
        if (zx < -128 || zx > 127) est |= AWEQ_ST_ZEROPOINT;
        if ((int)threadIdx.x <= rows_left) {
            if (zw < -128 || zw > 127) est |= AWEQ_ST_ZEROPOINT;
            s_scale[threadIdx.x] = (double)e_sx * (double)e_step;
            s_bias[threadIdx.x] = (double)e_bias;
            s_cn[threadIdx.x] = (unsigned)g.K * (unsigned)zx * (unsigned)zw - (unsigned)zx * (unsigned)e_rw;
            s_zw[threadIdx.x] = (unsigned)zw;
        } else if (QX == 0 && e_tok >= 0 && e_tok < kTokens) {
            s_rx[e_tok] = (unsigned)e_rw;
        }
    }
    __syncthreads();
    for (int e = threadIdx.x; e < kTiles * kWave; e += kThreads) {
        const int tile = e / kWave, l = e & (kWave - 1);
        const int64_t t = t0 + 16 * (tile / NT) + (l & 15), n = n0 + 16 * (tile % NT) + 4 * (l >> 4);
        const bool ok = t < g.T && n < g.N;     // N % 4 == 0: all four channels or none
        v4i o = {0, 0, 0, 0};
#pragma unroll
        for (int wv = 0; wv < kWaves; ++wv) o += *reinterpret_cast<const v4i*>(red + ((wv * kTiles + tile) * kWave + l) * 4);
        if (ok && g.out_i32) *reinterpret_cast<v4i*>(g.out_i32 + t * g.ldo + n) = o;
        if (ok && g.out_deq) {
            const int tl = 16 * (tile / NT) + (l & 15), nl = 16 * (tile % NT) + 4 * (l >> 4);
            const unsigned rs = QX != 0 ? (unsigned)s_rs[t] : s_rx[tl];
            float y[4];
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                const double div = (double)(int)((unsigned)o[c] + s_cn[nl + c] - s_zw[nl + c] * rs);
                y[c] = g.out_f16 ? (float)__builtin_fma(div, s_scale[nl + c], s_bias[nl + c]) : (float)(div * s_scale[nl + c] + s_bias[nl + c]);
            }
            if (g.out_f16) {
                typedef _Float16 h4 __attribute__((ext_vector_type(4)));
                *reinterpret_cast<h4*>(reinterpret_cast<_Float16*>(g.out_deq) + t * g.ldo + n) =
                    h4{(_Float16)y[0], (_Float16)y[1], (_Float16)y[2], (_Float16)y[3]};
            } else {
                *reinterpret_cast<Float4*>(reinterpret_cast<float*>(g.out_deq) + t * g.ldo + n) = Float4{{y[0], y[1], y[2], y[3]}};
            }
        }
        if (g.colsum_acc) {   // (uniform; every lane of a wavefront is here: kTiles * 64 is a multiple of it)
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                const long long s = group_allreduce<4>(ok ? (long long)o[c] : 0ll, OpAdd());
                if ((l & 15) == 0) s_col[tile / NT][16 * (tile % NT) + 4 * (l >> 4) + c] = s;
            }
        }
    }
    if (g.colsum_acc) {
        // one atomic per channel and workgroup (one per 16 tokens made a 2048 x 512 x 512 call take 16.4 us, 6.6 now)
        __syncthreads();
        const int c = threadIdx.x;
        if (c < 16 * NT && n0 + c < g.N) {
            long long s = 0;
#pragma unroll
            for (int i = 0; i < TT; ++i) s += s_col[i][c];
            atomicAdd(reinterpret_cast<unsigned long long*>(&g.colsum_acc[n0 + c]), (unsigned long long)s);
        }
    }
    raise_status(g.status, est);
}

// Token tiles ride on the grid's y dimension, at most 65535 to a launch: layers of up to 64 channels come here at any number of tokens
constexpr int kMaxGridY = 65535;
template <int TT, int NT, int D, int QX = 0, int TQ = 1>
static int launch_tile(GemmArgs g, hipStream_t st, QuantIn in = {})
{
    constexpr int kSums = kWaves * TT * NT * kWave * 16;   // partial sums; a launch that quantises has the tokens' codes behind them
    static_assert(QX == 0 || kSums + kQuantFewBytes <= 32768, "a launch that quantises stays below the LDS limit that has to be raised");
    const int lds = kSums + (QX != 0 ? (int)(g.T * panel_count(g.K) * kPanel) : 0);
    const void* fn = reinterpret_cast<const void*>(gemm_i8_few<TT, NT, D, QX, TQ>);
    int dev = 0, cus = 0;
    if (lds > 32768 && (device_cus(dev, cus) != AWEQ_OK || raise_lds_limit(fn, dev, lds) != AWEQ_OK)) return AWEQ_ERR_LAUNCH;
    void* args[] = {&g, &in};
    const int64_t tiles = cdiv(g.T, 16 * TT);
    for (int64_t first = 0; first < tiles; first += kMaxGridY) {
        g.run = (int)first;
        const unsigned gy = (unsigned)(tiles - first < kMaxGridY ? tiles - first : kMaxGridY);
        if (hipLaunchKernel(fn, dim3((unsigned)cdiv(g.N, 16 * NT), gy), dim3(kThreads), args, lds, st) != hipSuccess) return AWEQ_ERR_LAUNCH;
    }
    return launch_status();
}
}  // namespace few

// Tile by token count and channels.  Up to 32 tokens one row of workgroups covers them and the pass is a read of the
// weight: 16 channels per workgroup while they fill the chip 1.5 times over, then 32 (one token, us: 4096 x 4096 6.0 with
// 16 channels, 6.3 with 32; 16384 x 4096 14.0 / 12.8; 8192 x 8192 13.9 / 13.3).  Beyond that the tile whose rounds of 256
// workgroups, each weighted with its measured time at K = 8192, are cheapest (64 tokens, us, 32 x 32 / 32 x 64 / 64 x 64
// tiles: 4096 x 4096 7.6 / 9.3 / 12.2; 8192 x 8192 22.7 / 15.0 / 19.2; 16384 x 4096 23.3 / 24.2 / 14.8).
FewPlan plan_few(int64_t T, int64_t N)
{
    const bool wide = N > 6144;
    auto rounds = [&](int tt, int nt) { return (double)cdiv(cdiv(T, 16 * tt) * cdiv(N, 16 * nt), 256); };
    if (T <= 16) return wide ? FewPlan{1, 13.0 * rounds(1, 2)} : FewPlan{0, 13.0 * rounds(1, 2)};
    if (T <= 32) return wide ? FewPlan{3, 13.0 * rounds(2, 2)} : FewPlan{2, 13.0 * rounds(2, 2)};
    const double c22 = 13.0 * rounds(2, 2), c24 = 19.0 * rounds(2, 4), c44 = 22.0 * rounds(4, 4);
    if (c22 <= c24 && c22 <= c44) return FewPlan{3, c22};
    if (c24 <= c44) return FewPlan{4, c24};
    return FewPlan{5, c44};
}

int launch_gemm_i8_few_quant(const GemmArgs& g, const FewPlan& p, const QuantIn& in, bool f16, hipStream_t st)
{
#define AWEQ_FQ(NT, D, Q) (g.T == 1 ? few::launch_tile<1, NT, D, Q, 1>(g, st, in) : g.T == 2 ? few::launch_tile<1, NT, D, Q, 2>(g, st, in) : few::launch_tile<1, NT, D, Q, 4>(g, st, in))
    // Depth of the ring: three panels where nearly every compute unit has its one workgroup and a wavefront eight panels or more, four elsewhere, which
    // hold all panels of short rows and ask for more at a time where compute units are idle (us, buffers that change from call to call, 4 -> 3: one
    // token 4096 x 4096 6.17 -> 6.06, 4096 x 12288 12.3 -> 12.0, two tokens 3840 x 4096 6.55 -> 6.35, three tokens 4096 x 4096 7.35 -> 7.15, but one token
    // 4096 x 2048 4.22 -> 4.38, 2560 x 1536 3.69 -> 3.86, 3328 x 3072 5.1 -> 5.25, 2048 x 8192 6.9 -> 7.05, 1024 x 16384 9.65 -> 9.9, 6000 x 6144 8.75 -> 8.9)
    if (p.tile == 0 && g.N > 16 * 216 && g.N <= 16 * 256 && g.K >= 4096) return f16 ? AWEQ_FQ(1, 3, 1) : AWEQ_FQ(1, 3, 2);
    if (p.tile == 0) return f16 ? AWEQ_FQ(1, 4, 1) : AWEQ_FQ(1, 4, 2);
    return f16 ? AWEQ_FQ(2, 3, 1) : AWEQ_FQ(2, 3, 2);
#undef AWEQ_FQ
}

int launch_gemm_i8_few(const GemmArgs& g, const FewPlan& p, hipStream_t st)
{
    switch (p.tile) {
    case 0: return few::launch_tile<1, 1, 2>(g, st);
    case 1: return few::launch_tile<1, 2, 3>(g, st);
    case 2: return few::launch_tile<2, 1, 3>(g, st);
    case 3: return few::launch_tile<2, 2, 2>(g, st);
    case 4: return few::launch_tile<2, 4, 1>(g, st);
    default: return few::launch_tile<4, 4, 1>(g, st);
    }
}

}  // namespace aweq
