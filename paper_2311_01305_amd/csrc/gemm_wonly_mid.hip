// Weight-only forward for some hundred tokens: y = X_hat W~^T + b straight from the packed codes, where the few-token kernel
// would de-quantise every weight many times over and the tiled GEMM would leave most compute units without a tile.
//
// A workgroup of 8 wavefronts owns 64 WM tokens x 64 WN channels.  A stage is 64 WK values of K: wavefront (k, m, n) takes 64 of
// them for its 64 x 64 corner as 2 x 2 v_mfma_f32_32x32x16_f16 tiles, and the WK partial sums meet in LDS at the end, in a
// fixed order.  Activations, codes and (Step, Z) of a stage go through a ring of three LDS slots filled by LDS-DMA loads two
// stages ahead, one barrier a stage; 32 codes of a row are one 16-byte chunk of a slot in both formats (a three-dword
// load leaves the fourth dword of its lane's 16 bytes alone).  The weight operand is de-quantised in registers: a lane's
// 32 codes are its four operands of 8 values, lanes r and r + 32 hold values 0 .. 31 and 32 .. 63 of row r, and the
// activation operand enumerates K the same way.
//
// A stage of 64 x 128 x 256 takes 1.0 us: 0.7 us of loads (a compute unit takes 65 - 70 GB/s), 0.6 us of vector operations per
// SIMD (161 per wavefront, de-quantising for 64 tokens) and 0.5 us of MFMAs, interleaved word by word.  With 128 tokens
// per wavefront (128 x 256 tiles) the kernel was no faster than the de-quantising pass and the tiled GEMM.  us per
// call, INT4 groups of 128, without these tiles -> 64 x 128 / 128 x 128:
//   4096 x 4096    256 tokens 27.3 -> 22.5 / 37     512 tokens 50.3 -> 26.5 / 39    4096 x 11008   384 tokens 117 -> 55 / 95
//   11008 x 4096   128 tokens 40.4 -> 25 / 39       256 tokens 78.0 -> 48 / 42      768 tokens 118 -> 114 / 104
//   8192 x 8192    256 tokens 89.3 -> 48.6 / 76     384 tokens 98.5 -> 95 / 75
//   22016 x 8192   64 tokens 75.0 -> 50 / 79        128 tokens 140 -> 93 / 81       256 tokens 252 -> 140 / 164
#include "dequant.hpp"
#include "gemm_wonly_small.hpp"
#include <type_traits>

namespace aweq {
namespace wonly {
namespace mid {

typedef _Float16 v8h __attribute__((ext_vector_type(8)));
typedef float v16f __attribute__((ext_vector_type(16)));
typedef float v4f __attribute__((ext_vector_type(4)));

constexpr int kThreads = 512;

template <int WM, int WN, int WK>
struct Tile {
    static_assert(WM * WN * WK == 8, "eight wavefronts");
    static constexpr int kM = 64 * WM, kN = 64 * WN, kK = 64 * WK;
    static constexpr int kRowX = kK * 2, kRowC = kK / 2;               // slot bytes of a row of activations, of codes
    static constexpr int kSegs = kK / 128;                             // (Step, Z) pairs per row
    static constexpr int kX = kM * kRowX, kC = kN * kRowC, kS = kN * kSegs * 4;
    static constexpr int kSlot = kX + kC + 2 * kS;
    static constexpr int kSlots = 3;
    static constexpr int kLoadsX = kX / 8192, kLoadsC = kC / 8192, kLoads = kLoadsX + kLoadsC + 1;
    static constexpr int kSums = 128 * 1024;                           // partial sums: 16 KiB per wavefront
    static constexpr int kLds = kSlots * kSlot > kSums ? kSlots * kSlot : kSums;
    static_assert(kLds <= 160 * 1024, "LDS");
};

// chunk swizzles: rows of codes sit 64 or 128 bytes apart (as in the int8 kernels and the tiled kernel)
template <int ROW> __device__ __forceinline__ int code_swz(int r)
{
    return ROW == 64 ? (r >> 2) & 3 : ((((r >> 1) & 3) << 1) | (((r >> 3) ^ r) & 1));
}

// LDS-DMA loads the compiler does not track: lane i's bytes land at lds_addr + 16 i (4 i: one dword)
template <int DWORDS>
__device__ __forceinline__ void dma(const char* sbase, uint32_t voff, uint32_t lds_addr)
{
    if constexpr (DWORDS == 4) asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" ::"s"(lds_addr), "v"(voff), "s"(sbase) : "memory");
    else if constexpr (DWORDS == 3) asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx3 %1, %2" ::"s"(lds_addr), "v"(voff), "s"(sbase) : "memory");
    else asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dword %1, %2" ::"s"(lds_addr), "v"(voff), "s"(sbase) : "memory");
}
template <int N>
__device__ __forceinline__ void wait_vm()
{
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
}

template <int BITS, int WM, int WN, int WK, bool OUT_F16>
__global__ __launch_bounds__(kThreads) void gemm_mid_kernel(SmallArgs g, int tiles_m, int tiles_n, int run)
{
    using TL = Tile<WM, WN, WK>;
    extern __shared__ __attribute__((aligned(1024))) char lds[];
    const int tid = threadIdx.x, lane = tid & (kWave - 1);
    const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);
    const int wk = wave / (WM * WN), wm = wave / WN % WM, wn = wave % WN;

    // ids are dealt round-robin to the XCDs: each XCD takes an equal run of the tiles, token tiles fastest, so that a row of
    // codes is read by one or two XCDs only
    const int l = (int)(blockIdx.x % kXcdCount) * run + (int)(blockIdx.x / kXcdCount);
    if (l >= tiles_m * tiles_n) return;
    const int64_t m0 = (int64_t)(l % tiles_m) * TL::kM, n0 = (int64_t)(l / tiles_m) * TL::kN;
    const int K = (int)g.K, ns = (K + TL::kK - 1) / TL::kK;
    const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char*)lds;

    // this thread's share of the epilogue: four channels, every kRowStep-th token; the bias is requested ahead of the operands
    constexpr int kRowThreads = TL::kN / 4, kRowStep = kThreads / kRowThreads, kRows = TL::kM / kRowStep;
    const int ec = tid % kRowThreads, er = tid / kRowThreads;
    const int64_t n = n0 + ec * 4;
    const bool n_ok = n < g.N;     // N % 4 == 0: all four channels or none
    v4f bs = {0.f, 0.f, 0.f, 0.f};
    if (g.bias && n_ok) bs = *reinterpret_cast<const v4f*>(g.bias + n);

    // Loads of a stage, per wavefront: kLoadsX KiB of activations, kLoadsC KiB of codes, 64 scales.  Offsets of this lane's
    // rows from the tile's first; rows past the edge re-read the last valid row, their results are never stored.
    constexpr int kChunksX = TL::kRowX / 16, kChunksC = TL::kRowC / 16;
    uint32_t xrow[TL::kLoadsX], xcol[TL::kLoadsX], crow[TL::kLoadsC], ccol[TL::kLoadsC];
#pragma unroll
    for (int q = 0; q < TL::kLoadsX; ++q) {
        const int e = (wave * TL::kLoadsX + q) * kWave + lane, row = e / kChunksX;
        xrow[q] = (uint32_t)min((int64_t)row, g.T - 1 - m0) * (uint32_t)g.ldx;
        xcol[q] = (uint32_t)((e % kChunksX) ^ (row & 15)) * 8;
    }
    const uint32_t code_pitch = (uint32_t)(K >> 3) * BITS;
#pragma unroll
    for (int q = 0; q < TL::kLoadsC; ++q) {
        const int e = (wave * TL::kLoadsC + q) * kWave + lane, row = e / kChunksC;
        crow[q] = (uint32_t)min((int64_t)row, g.N - 1 - n0) * code_pitch;
        ccol[q] = (uint32_t)((e % kChunksC) ^ code_swz<TL::kRowC>(row)) * 32;
    }
    // scales: unit (array, segment, 64 rows); fewer than eight units: the same 256 bytes are loaded twice
    constexpr int kUnitsS = 2 * TL::kSegs * TL::kN / kWave;
    const int su = wave % kUnitsS, sarr = su / (kUnitsS / 2), sseg = su % (kUnitsS / 2) / (TL::kN / kWave), srows = su % (TL::kN / kWave) * kWave;
    const uint32_t soff = (uint32_t)min((int64_t)(srows + lane), g.N - 1 - n0) * g.scale_pitch * 4;
    const char* const sbase = (sarr ? reinterpret_cast<const char*>(g.zero) : reinterpret_cast<const char*>(g.step)) + n0 * g.scale_pitch * 4;
    const char* const xbase = reinterpret_cast<const char*>(g.X + m0 * g.ldx);
    const char* const cbase = reinterpret_cast<const char*>(g.codes) + n0 * code_pitch;
    // load q of a stage: activations, codes, scales
    auto issue = [&](int s, int q) {
        const uint32_t slot = lds0 + (uint32_t)(s % TL::kSlots) * TL::kSlot;
        const int k0 = s * TL::kK;
        const uint32_t left = (uint32_t)(K - k0);   // columns past K: the last valid ones again, not multiplied
        if (q < TL::kLoadsX) {
            dma<4>(xbase + (int64_t)k0 * 2, (xrow[q] + min(xcol[q], left - 8)) * 2, slot + (uint32_t)(wave * TL::kLoadsX + q) * 1024);
        } else if (q < TL::kLoadsX + TL::kLoadsC) {
            const int c = q - TL::kLoadsX;
            dma<BITS>(cbase + (int64_t)(k0 / 8) * BITS, crow[c] + min(ccol[c], left - 32) / 8 * BITS, slot + TL::kX + (uint32_t)(wave * TL::kLoadsC + c) * 1024);
        } else {
            const int ks = min(k0 + sseg * 128, K - 64);
            dma<1>(sbase + (int64_t)__umulhi((uint32_t)ks >> 4, g.group_magic) * 4, soff, slot + TL::kX + TL::kC + (uint32_t)su * 256);
        }
    };

    const int fr_row = lane & 31, fr_half = lane >> 5;
    const int coff = TL::kX + (wn * 64 + fr_row) * TL::kRowC + (((wk * 2 + fr_half) ^ code_swz<TL::kRowC>(fr_row)) * 16);
    const int soff_r = TL::kX + TL::kC + ((wk / 2) * TL::kN + wn * 64 + fr_row) * 4;
    const int xoff = (wm * 64 + fr_row) * TL::kRowX, xchunk = wk * 8 + fr_half * 4, xswz = fr_row & 15;

    v16f acc[2][2];
    bool packed = true;   // no zero point so far was outside the packed path
    // MORE: stage s + 2 is requested between the multiplications (a load instruction waits until the address unit takes it)
    auto stage = [&](int s, auto packed_c, auto more_c) {
        const char* const st = lds + (s % TL::kSlots) * TL::kSlot;
        v4i x[2][2];   // of the K-step at hand and the next
        RawCodes<BITS> c[2];
        Scale<BITS> sc[2];
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            const v4i cw = *reinterpret_cast<const v4i*>(st + coff + j * 32 * TL::kRowC);
#pragma unroll
            for (int e = 0; e < (BITS == 4 ? 4 : 3); ++e) c[j].w[e] = (uint32_t)cw[e];
            sc[j].set(*reinterpret_cast<const float*>(st + soff_r + j * 128), *reinterpret_cast<const int32_t*>(st + soff_r + TL::kS + j * 128));
            packed = packed && sc[j].packed;
        }
        auto fetch_x = [&](int d) {
#pragma unroll
            for (int i = 0; i < 2; ++i) x[d & 1][i] = *reinterpret_cast<const v4i*>(st + xoff + i * 32 * TL::kRowX + (((xchunk + d) ^ xswz) * 16));
        };
        fetch_x(0);
        auto operand = [&](int e) {   // words in the order d, j
            const int d = e >> 1, j = e & 1;
            uint32_t cw;
            if constexpr (BITS == 4) cw = c[j].w[d];
            else cw = fields3(c[j], d);
            if constexpr (decltype(packed_c)::value) return dequant_word_natural<BITS>(cw, sc[j]);
            else {
                uint32_t o[4];
                dequant_word_any<BITS>(cw, sc[j], o);
                return natural_order(o);
            }
        };
        v4i w[2];
        w[0] = operand(0);
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            __builtin_amdgcn_sched_barrier(0);
            if constexpr (decltype(more_c)::value) {
                if (e < TL::kLoads) issue(s + TL::kSlots - 1, e);
            }
            const int d = e >> 1, j = e & 1;
            if (j == 0 && d < 3) fetch_x(d + 1);
            auto mul = [&](int i) {
                acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(v8h, w[e & 1]), __builtin_bit_cast(v8h, x[d & 1][i]), acc[i][j], 0, 0, 0);
            };
            mul(0);
            if (e < 7) w[(e + 1) & 1] = operand(e + 1);
            mul(1);
        }
    };
    auto run_stages = [&](auto packed_c) {
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int j = 0; j < 2; ++j)
#pragma unroll
                for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.0f;
        for (int s = 0; s < TL::kSlots - 1 && s < ns; ++s)
#pragma unroll
            for (int q = 0; q < TL::kLoads; ++q) issue(s, q);
        static_assert(TL::kLoads <= 8, "one load per step of a stage");
        // stage s has landed for this wavefront (the one after it may be out), its reads of stage s - 1 are done; after the
        // barrier that holds for every wavefront, and stage s + 2 can take the slot of stage s - 1
        int s = 0;
        for (; s + TL::kSlots - 1 < ns; ++s) {
            wait_vm<TL::kLoads>();
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
            __builtin_amdgcn_s_barrier();
            stage(s, packed_c, std::true_type{});
        }
        for (; s < ns; ++s) {
            if (s + 1 < ns) wait_vm<TL::kLoads>(); else wait_vm<0>();
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
            __builtin_amdgcn_s_barrier();
            if (s * TL::kK + wk * 64 < K) stage(s, packed_c, std::false_type{});
        }
    };
    run_stages(std::true_type{});
    // a zero point outside the packed path (rare): the tile again through binary32, rather than a branch in every stage
    if (__syncthreads_or(packed ? 0 : 1)) run_stages(std::false_type{});
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    __builtin_amdgcn_s_barrier();   // every wavefront is done with the ring

    // register v of lane l in sub-tile (i, j) is token 32 i + l % 32 and channel 32 j + 8 (v / 4) + 4 (l / 32) + v % 4 of the
    // wavefront's corner: rows of 256 bytes, 16-byte chunks XOR swizzled
    char* const mine = lds + wave * 16384;
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int t = 32 * i + fr_row;
                *reinterpret_cast<v4f*>(mine + t * 256 + (((8 * j + 2 * q + fr_half) ^ (t & 15)) * 16)) =
                    v4f{acc[i][j][4 * q], acc[i][j][4 * q + 1], acc[i][j][4 * q + 2], acc[i][j][4 * q + 3]};
            }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < kRows; ++i) {
        const int r = er + i * kRowStep;
        const int64_t t = m0 + r;
        if (t >= g.T || !n_ok) continue;
        v4f o = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int k = 0; k < WK; ++k)
            o += *reinterpret_cast<const v4f*>(lds + ((k * WM + r / 64) * WN + ec / 16) * 16384 + (r & 63) * 256 + (((ec & 15) ^ (r & 15)) * 16));
        o += bs;
        if constexpr (OUT_F16) {
            typedef _Float16 h4 __attribute__((ext_vector_type(4)));
            *reinterpret_cast<h4*>(reinterpret_cast<_Float16*>(g.out) + t * g.ldo + n) = h4{(_Float16)o[0], (_Float16)o[1], (_Float16)o[2], (_Float16)o[3]};
        } else {
            *reinterpret_cast<v4f*>(reinterpret_cast<float*>(g.out) + t * g.ldo + n) = o;
        }
    }
}

template <int BITS, int WM, int WN, int WK>
static int launch_tile(SmallArgs g, bool out_f16, hipStream_t st)
{
    using TL = Tile<WM, WN, WK>;
    int tiles_m = (int)cdiv(g.T, TL::kM), tiles_n = (int)cdiv(g.N, TL::kN);
    int run = (int)cdiv((int64_t)tiles_m * tiles_n, kXcdCount);
    const void* fn = out_f16 ? reinterpret_cast<const void*>(gemm_mid_kernel<BITS, WM, WN, WK, true>)
                             : reinterpret_cast<const void*>(gemm_mid_kernel<BITS, WM, WN, WK, false>);
    int dev = 0, cus = 0;
    if (device_cus(dev, cus) != AWEQ_OK || raise_lds_limit(fn, dev, TL::kLds) != AWEQ_OK) return AWEQ_ERR_LAUNCH;
    void* args[] = {&g, &tiles_m, &tiles_n, &run};
    if (hipLaunchKernel(fn, dim3((unsigned)(run * kXcdCount)), dim3(kThreads), args, TL::kLds, st) != hipSuccess) return AWEQ_ERR_LAUNCH;
    return launch_status();
}

}  // namespace mid

// the tile whose rounds of 256 workgroups are cheaper (us at K = 8192, as in plan_small)
MidPlan plan_mid(int64_t T, int64_t N)
{
    auto rounds = [&](int bm, int bn) { return (double)cdiv(cdiv(T, bm) * cdiv(N, bn), 256); };
    const double c12 = 47.0 * rounds(64, 128), c22 = 78.0 * rounds(128, 128);
    return c12 <= c22 ? MidPlan{false, c12} : MidPlan{true, c22};
}

int launch_mid(const SmallArgs& g, int bits, const MidPlan& p, bool out_f16, hipStream_t st)
{
    if (bits == 4) return p.square ? mid::launch_tile<4, 2, 2, 2>(g, out_f16, st) : mid::launch_tile<4, 1, 2, 4>(g, out_f16, st);
    return p.square ? mid::launch_tile<3, 2, 2, 2>(g, out_f16, st) : mid::launch_tile<3, 1, 2, 4>(g, out_f16, st);
}

}  // namespace wonly
}  // namespace aweq
