// Stage 4b for some hundred tokens: the int8 GEMM when 128 x 256 tiles leave most compute units without one.
//
// A workgroup of 8 wavefronts owns 64 WM tokens x 64 WN channels.  A stage is WK panels of K (64 bytes each): wavefront
// (k, m, n) multiplies panel k of it for its 64 x 64 corner as 2 x 2 v_mfma_i32_32x32x32_i8 tiles, so that a small tile still has
// all eight wavefronts at 1 KiB of LDS reads per MFMA, and the WK partial sums meet in LDS at the end.  Stages go through
// a ring of kSlots LDS slots filled by LDS-DMA loads, kSlots - 1 stages ahead, one barrier a stage; slots, swizzle and operand
// order are the tiled kernel's.
//
// Bound by what a compute unit can load: 65 - 70 GB/s of operands each whatever the tile (reading a stage's fragments
// ahead of the barrier, which overlaps them with the stage before, gains nothing).  us per call, binary16 output, without these
// tiles (64- and 128-token tiles of the other kernels) -> 64 x 128 / 128 x 128:
//   4096 x 4096    512 tokens 26.1 -> 17.9 / 24.6     4096 x 11008   384 tokens 68.5 -> 39.1 / 52.9   768 tokens 68.6 -> 75.2 / 54.4
//   11008 x 4096   128 tokens 33.1 -> 20.8 / 26.3     192 tokens 30.8 -> 34.7 / 26.2
//   8192 x 8192    256 tokens 56.0 -> 33.5 / 42.6     512 tokens 55.2 -> 63.3 / 46.8
//   22016 x 8192   128 tokens 62.9 -> 67.2 / 47.4
#include "gemm_i8.hpp"

namespace aweq {
namespace mid {

typedef int v4i __attribute__((ext_vector_type(4)));
typedef int v16i __attribute__((ext_vector_type(16)));

constexpr int kThreads = 512;

template <int WM, int WN, int WK>
struct Tile {
    static_assert(WM * WN * WK == 8, "eight wavefronts");
    static constexpr int kM = 64 * WM, kN = 64 * WN;
    static constexpr int kPanelBytes = (kM + kN) * kPanel;             // one panel: the activation rows, then the weight rows
    static constexpr int kSlot = WK * kPanelBytes;
    static constexpr int kSlots = 160 * 1024 / kSlot >= 4 ? 4 : 160 * 1024 / kSlot;
    static constexpr int kLoads = kSlot / 1024 / 8;                     // load instructions per wavefront and stage
    static constexpr int kSums = 128 * 1024;                            // partial sums: 16 KiB per wavefront
    static constexpr int kLds = kSlots * kSlot > kSums ? kSlots * kSlot : kSums;
};

// chunk swizzle for 64-byte slot rows (as in the tiled kernel)
__device__ __forceinline__ int f4(int r) { return (r >> 2) & 3; }

// LDS-DMA load the compiler does not track: lane i's 16 bytes land at lds_addr + 16 i
__device__ __forceinline__ void dma16(const int8_t* sbase, uint32_t voff, uint32_t lds_addr)
{
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" ::"s"(lds_addr), "v"(voff), "s"(sbase) : "memory");
}
template <int N>
__device__ __forceinline__ void wait_vm()
{
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
}

// QUANT: the epilogue also quantises the binary16 output for the next layer (aweq_w8a8_gemm_fused without statistics)
template <int WM, int WN, int WK, bool QUANT>
__global__ __launch_bounds__(kThreads) void gemm_i8_mid(GemmArgs g)
{
    using TL = Tile<WM, WN, WK>;
    extern __shared__ __attribute__((aligned(1024))) char lds[];
    const int tid = threadIdx.x, lane = tid & (kWave - 1);
    const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);
    const int wk = wave / (WM * WN), wm = wave / WN % WM, wn = wave % WN;

    // ids are dealt round-robin to the XCDs: each XCD takes an equal run of the tiles, token tiles fastest, so that a weight
    // row is read by one or two XCDs only
    const int l = (int)(blockIdx.x % kXcdCount) * g.run + (int)(blockIdx.x / kXcdCount);
    if (l >= g.tiles_m * g.tiles_n) return;
    const int64_t m0 = (int64_t)(l % g.tiles_m) * TL::kM, n0 = (int64_t)(l / g.tiles_m) * TL::kN;

    const int np = (int)panel_count(g.K), ns = (np + WK - 1) / WK;
    const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char*)lds;

    // this thread's share of the epilogue: four channels, every kRowStep-th token; what it needs from memory is requested
    // ahead of the operands
    constexpr int kRowThreads = TL::kN / 4, kRowStep = kThreads / kRowThreads, kRows = TL::kM / kRowStep;
    const int ec = tid % kRowThreads, er = tid / kRowThreads;
    const int64_t n = n0 + ec * 4;
    const bool n_ok = n < g.N;     // N % 4 == 0: all four channels or none
    int zx = 0, zw[4] = {0, 0, 0, 0}, rw[4] = {0, 0, 0, 0}, rsx[kRows];
    float sxf = 0.f, sw[4] = {0.f, 0.f, 0.f, 0.f}, bs[4] = {0.f, 0.f, 0.f, 0.f};
    const bool deq = QUANT || g.out_deq;
    if (deq) {
        zx = *g.act_zero - 128;
        sxf = *g.act_step;
#pragma unroll
        for (int c = 0; c < 4; ++c)
            if (n_ok) {
                const int64_t pi = g.w_per_tensor ? 0 : n + c;
                sw[c] = g.step_w[pi];
                zw[c] = g.zero_w[pi] - 128;
                rw[c] = g.rowsum_w[n + c];
                if (g.bias) bs[c] = g.bias[n + c];
            }
#pragma unroll
        for (int i = 0; i < kRows; ++i) rsx[i] = g.rowsum_x[min(m0 + er + i * kRowStep, g.T - 1)];
    }

    // load q of this wavefront brings 16 rows of one panel of the stage: unit wave kLoads + q of (panel, 16-row group)
    constexpr int kGroups = 4 * (WM + WN);
    uint32_t voff[TL::kLoads];
#pragma unroll
    for (int q = 0; q < TL::kLoads; ++q) {
        const int grp = (wave * TL::kLoads + q) % kGroups, sub = lane >> 2;
        // rows past the edge re-read the last valid row; their results are never stored
        const int row = grp < 4 * WM ? (int)min((int64_t)(grp * 16 + sub), g.T - 1 - m0) : (int)min((int64_t)((grp - 4 * WM) * 16 + sub), g.N - 1 - n0);
        voff[q] = (uint32_t)(row * kPanel + ((lane & 3) ^ f4(sub)) * 16);
    }
    const int8_t* const baseA = g.A + m0 * kPanel;
    const int8_t* const baseB = g.B + n0 * kPanel;
    auto issue = [&](int s) {
        const uint32_t slot = lds0 + (uint32_t)(s % TL::kSlots) * TL::kSlot;
#pragma unroll
        for (int q = 0; q < TL::kLoads; ++q) {
            const int unit = wave * TL::kLoads + q;
            const int64_t p = min(s * WK + unit / kGroups, np - 1);   // (panels past the last one re-read it: they are not multiplied)
            const bool a = unit % kGroups < 4 * WM;
            dma16((a ? baseA : baseB) + p * ((a ? g.T : g.N) * kPanel), voff[q], slot + (uint32_t)unit * 1024);
        }
    };

    const int fr_row = lane & 31, fr_half = lane >> 5;
    int offA[2], offB[2];
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) {
        const int chunk = ((ks * 2 + fr_half) ^ f4(fr_row)) * 16;
        offA[ks] = wk * TL::kPanelBytes + (wm * 64 + fr_row) * kPanel + chunk;
        offB[ks] = wk * TL::kPanelBytes + (TL::kM + wn * 64 + fr_row) * kPanel + chunk;
    }

    v16i acc[2][2];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[i][j][v] = 0;

    for (int s = 0; s < TL::kSlots - 1 && s < ns; ++s) issue(s);
    for (int s = 0; s < ns; ++s) {
        // stage s has landed for this wavefront (stages after it may be out), its reads of stage s - 1 are done; after the
        // barrier that holds for every wavefront, and stage s + kSlots - 1 can take the slot of stage s - 1
        const int newer = min(TL::kSlots - 2, ns - 1 - s);
        if (newer == 0) wait_vm<0>();
        else if (newer == 1) wait_vm<TL::kLoads>();
        else wait_vm<2 * TL::kLoads>();
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        __builtin_amdgcn_s_barrier();
        if (s + TL::kSlots - 1 < ns) issue(s + TL::kSlots - 1);
        if (s * WK + wk < np) {
            const char* const st = lds + (s % TL::kSlots) * TL::kSlot;
            v4i a[2][2], b[2][2];
#pragma unroll
            for (int ks = 0; ks < 2; ++ks)
#pragma unroll
                for (int i = 0; i < 2; ++i) {
                    a[ks][i] = *reinterpret_cast<const v4i*>(st + offA[ks] + i * 32 * kPanel);
                    b[ks][i] = *reinterpret_cast<const v4i*>(st + offB[ks] + i * 32 * kPanel);
                }
#pragma unroll
            for (int ks = 0; ks < 2; ++ks)
#pragma unroll
                for (int i = 0; i < 2; ++i)
#pragma unroll
                    for (int j = 0; j < 2; ++j) acc[i][j] = __builtin_amdgcn_mfma_i32_32x32x32_i8(b[ks][j], a[ks][i], acc[i][j], 0, 0, 0);
        }
    }
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    __builtin_amdgcn_s_barrier();   // every wavefront is done with the ring

    // register v of lane l in sub-tile (i, j) is token 32 i + l % 32 and channel 32 j + 8 (v / 4) + 4 (l / 32) + v % 4 of the
    // wavefront's corner: rows of 256 bytes, 16-byte chunks XOR swizzled
    {
        char* const mine = lds + wave * 16384;
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int j = 0; j < 2; ++j)
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const int t = 32 * i + fr_row;
                    *reinterpret_cast<v4i*>(mine + t * 256 + (((8 * j + 2 * q + fr_half) ^ (t & 15)) * 16)) =
                        v4i{acc[i][j][4 * q], acc[i][j][4 * q + 1], acc[i][j][4 * q + 2], acc[i][j][4 * q + 3]};
                }
    }
    __syncthreads();

    uint32_t est = 0;
    unsigned cn[4] = {0, 0, 0, 0};
    double scale[4] = {0, 0, 0, 0};
    if (deq) {
        // the tiled kernel's arithmetic: the integer part in wrap-around 32 bits, scaled and shifted in fp64
        if (zx < -128 || zx > 127) est |= AWEQ_ST_ZEROPOINT;
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            if (zw[c] < -128 || zw[c] > 127) est |= AWEQ_ST_ZEROPOINT;
            cn[c] = (unsigned)g.K * (unsigned)zx * (unsigned)zw[c] - (unsigned)zx * (unsigned)rw[c];
            scale[c] = (double)sxf * (double)sw[c];
        }
    }
    // the next layer's quantizer, as in the tiled kernel's fused epilogue
    float nis[4] = {1.f, 1.f, 1.f, 1.f};
    ActParams np_ = {};
    bool nscreen = false;
    if constexpr (QUANT) {
        np_ = quot_params(*g.next_step, *g.next_zero);
        nscreen = np_.screen;
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            if (n_ok) nis[c] = g.next_inv_s[n + c];
            nscreen = nscreen && 65600.0f * fabsf(nis[c]) * np_.rstep < 16777216.0f;
        }
    }
    long long csum[4] = {0, 0, 0, 0}, qsum[4] = {0, 0, 0, 0};
    int rs_kept = 0;   // row sum of the codes of this thread's ec-th token
#pragma unroll
    for (int i = 0; i < kRows; ++i) {
        const int r = er + i * kRowStep;
        const int64_t t = m0 + r;
        const bool ok = t < g.T && n_ok;
        v4i o = {0, 0, 0, 0};
        if (ok) {
#pragma unroll
            for (int k = 0; k < WK; ++k) {
                const char* const part = lds + ((k * WM + r / 64) * WN + ec / 16) * 16384;
                o += *reinterpret_cast<const v4i*>(part + (r & 63) * 256 + (((ec & 15) ^ (r & 15)) * 16));
            }
        }
        int rs = 0;
        if (!QUANT && ok && g.out_i32) *reinterpret_cast<v4i*>(g.out_i32 + t * g.ldo + n) = o;
        if (ok && deq) {
            typedef _Float16 h4 __attribute__((ext_vector_type(4)));
            float y[4];
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                const double div = (double)(int)((unsigned)o[c] + cn[c] - (unsigned)zw[c] * (unsigned)rsx[i]);
                y[c] = QUANT || g.out_f16 ? (float)__builtin_fma(div, scale[c], (double)bs[c]) : (float)(div * scale[c] + (double)bs[c]);
                if (QUANT && g.act == 1) y[c] = fmaxf(y[c], 0.0f);
            }
            const h4 oh = {(_Float16)y[0], (_Float16)y[1], (_Float16)y[2], (_Float16)y[3]};
            if (QUANT || g.out_f16) {
                if (g.out_deq) *reinterpret_cast<h4*>(reinterpret_cast<_Float16*>(g.out_deq) + t * g.ldo + n) = oh;
            } else {
                *reinterpret_cast<Float4*>(reinterpret_cast<float*>(g.out_deq) + t * g.ldo + n) = Float4{{y[0], y[1], y[2], y[3]}};
            }
            if constexpr (QUANT) {
                uint32_t w = 0;
                float u[4], dmax = 0.0f;
#pragma unroll
                for (int c = 0; c < 4; ++c) {
                    const float a = __builtin_fmaf((float)oh[c], nis[c], 0.0f);
                    const float q = __builtin_fmaf(a, np_.rstep, (float)np_.zero);
                    u[c] = rintf(q);
                    dmax = fmaxf(dmax, fabsf(q - u[c]));
                }
                if (!nscreen || dmax > np_.thr) {
#pragma unroll
                    for (int c = 0; c < 4; ++c) u[c] = (float)quant_div((float)oh[c] * nis[c], np_.step, np_.zero, 255, est);
                }
#pragma unroll
                for (int c = 0; c < 4; ++c) {
                    u[c] = __builtin_amdgcn_fmed3f(u[c], 0.0f, 255.0f);
                    qsum[c] += (int)u[c] - 128;
                    w = __builtin_amdgcn_cvt_pk_u8_f32(u[c], c, w);
                }
                w ^= 0x80808080u;
                rs = __builtin_amdgcn_sdot4((int)w, 0x01010101, 0, false);
                *reinterpret_cast<uint32_t*>(g.yq + panel_offset(g.T, t, n)) = w;
            }
        } else if (QUANT && t < g.T && (n & ~(int64_t)(kPanel - 1)) < g.N) {
            *reinterpret_cast<uint32_t*>(g.yq + panel_offset(g.T, t, n)) = 0u;   // zero fill of the last panel
        }
        if constexpr (QUANT) {
            static_assert(kRowThreads == 32 && kRows <= 32, "a token's channels sit in half a wavefront");
            rs = group_allreduce<5>(rs, OpAdd());
            rs_kept = ec == i ? rs : rs_kept;
        }
#pragma unroll
        for (int c = 0; c < 4; ++c) csum[c] += o[c];
    }
    if (QUANT && g.rowsum_y && ec < kRows) {
        const int64_t t = m0 + er + ec * kRowStep;
        if (t < g.T) atomicAdd(&g.rowsum_y[t], rs_kept);
    }
    // sums over the tokens: threads with the same channels are lanes 32 apart, then the wavefronts
    auto add_columns = [&](long long v[4], long long* dst) {
        __syncthreads();
        long long* const red = reinterpret_cast<long long*>(lds);   // [wavefront][channel]
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            v[c] += partner<5>(v[c]);
            if (lane < kRowThreads) red[wave * TL::kN + lane * 4 + c] = v[c];
        }
        __syncthreads();
        for (int ch = tid; ch < TL::kN; ch += kThreads) {
            long long sum = 0;
#pragma unroll
            for (int w = 0; w < 8; ++w) sum += red[w * TL::kN + ch];
            if (n0 + ch < g.N) atomicAdd(reinterpret_cast<unsigned long long*>(&dst[n0 + ch]), (unsigned long long)sum);
        }
    };
    if (g.colsum_acc) add_columns(csum, g.colsum_acc);
    if (QUANT && g.colsum_yq) add_columns(qsum, g.colsum_yq);
    raise_status(g.status, est);
}

template <int WM, int WN, int WK, bool QUANT>
static int launch_tile(GemmArgs g, hipStream_t st)
{
    using TL = Tile<WM, WN, WK>;
    g.tiles_m = (int)cdiv(g.T, TL::kM);
    g.tiles_n = (int)cdiv(g.N, TL::kN);
    g.run = (int)cdiv((int64_t)g.tiles_m * g.tiles_n, kXcdCount);
    const void* fn = reinterpret_cast<const void*>(gemm_i8_mid<WM, WN, WK, QUANT>);
    int dev = 0, cus = 0;
    if (device_cus(dev, cus) != AWEQ_OK || raise_lds_limit(fn, dev, TL::kLds) != AWEQ_OK) return AWEQ_ERR_LAUNCH;
    void* args[] = {&g};
    if (hipLaunchKernel(fn, dim3((unsigned)(g.run * kXcdCount)), dim3(kThreads), args, TL::kLds, st) != hipSuccess) return AWEQ_ERR_LAUNCH;
    return launch_status();
}

}  // namespace mid

// the tile whose rounds of 256 workgroups are cheaper (us at K = 8192, as in the plans of the other forms: one round of 64 x 128
// tiles was measured at 32.5, of 128 x 128 tiles at 42.5).  Rounds after the first come dearer, their workgroups do not overlap
// the end of one tile with the start of the next as the persistent form's do: four of 128 x 128 tiles against three of the persistent
// 128 x 256 ones 195 / 169 us (6581 tokens 2432 x 7616), 68.7 / 54.4 (7173 tokens 2104 x 1600)
MidPlan plan_mid(int64_t T, int64_t N)
{
    auto rounds = [&](int bm, int bn) { return (double)cdiv(cdiv(T, bm) * cdiv(N, bn), 256); };
    const double r22 = rounds(128, 128), c12 = 32.0 * rounds(64, 128), c22 = (r22 >= 4.0 ? 48.0 : 43.0) * r22;
    return c12 <= c22 ? MidPlan{false, c12} : MidPlan{true, c22};
}

int launch_gemm_i8_mid(const GemmArgs& g, const MidPlan& p, hipStream_t st)
{
    if (g.yq) return p.square ? mid::launch_tile<2, 2, 2, true>(g, st) : mid::launch_tile<1, 2, 4, true>(g, st);
    return p.square ? mid::launch_tile<2, 2, 2, false>(g, st) : mid::launch_tile<1, 2, 4, false>(g, st);
}

}  // namespace aweq
