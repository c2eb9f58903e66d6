// Stage 4b: W8A8 GEMM  acc[t,n] = sum_k xq[t,k] wq[n,k]  (int8 x int8 -> int32) on the
// gfx950 matrix cores, with the epilogues the calibration path needs: raw int32 output,
// de-quantised output, and the per-output-channel sum over tokens (int64) that feeds the
// bias correction of Sec. 3.3.
//
// Both operands arrive in the K-panel layout (64-byte panels of K, rows back to back inside a
// panel, zero fill past K): the 256 rows x 64 bytes an output tile needs of one panel are one
// contiguous 16 KiB block, every cache line is used whole, and any K % 8 == 0 works.
//
// MFMA-bound by design, load-round-trip-bound in practice, which fixes the structure.  Two kernels:
//  - gemm_i8_fast (N % 4 == 0, 16-byte aligned outputs): one workgroup of 8 wavefronts
//    (two per SIMD) owns a 256 x 256 output tile, each wavefront 128 (t) x 64 (n) of it as
//    4 x 2 v_mfma_i32_32x32x32_i8 tiles; a lane's MFMA operand is 16 consecutive bytes of one
//    row.  Half-stages of one panel (256 rows x 64 bytes per operand, 32 KiB) go through a ring
//    of four LDS slots filled by LDS-DMA loads (global_load_lds_dwordx4, no staging registers),
//    three half-stages ahead of the one being multiplied: the round trip of a load under
//    load (about 1.5 us when part of it misses the L2) is longer than the 0.5 - 1 us a stage of
//    MFMAs lasts, so a two-buffer scheme stalls on every stage whatever the issue order.
//    The slots are XOR swizzled by choosing which 16-byte chunk each lane fetches; loads, LDS
//    fragment reads for the next K-step and MFMAs are interleaved by hand.  The MFMA is
//    issued with the weight fragment as its first operand, so a lane ends up with four
//    consecutive n of one token: 16-byte output stores.  A second form has tiles of 128 x 256
//    (wavefronts of 64 x 64, a ring of five 24 KiB slots) for calls with few tiles.
//  - gemm_i8_generic (any N, any alignment): 4 wavefronts, half-stages through registers;
//    slower, used for shapes the fast kernel does not take.
// Workgroups are numbered so that the ones resident on one XCD (which share an L2) form a
// compact patch of the output.
#include "gemm_i8.hpp"
#include "quant_act.hpp"
#include "row_reduce.hpp"
#include <type_traits>

namespace aweq {

typedef int v4i __attribute__((ext_vector_type(4)));
typedef int v16i __attribute__((ext_vector_type(16)));

constexpr int kGemmThreads = 256;
constexpr int BM = 256, BN = 256, BK = 64;
constexpr int kChunksPerRow = BK / 16;                       // 16-byte chunks per tile row
constexpr int kTileBytes = BM * BK;                          // 16 KiB per operand tile
constexpr int kLoadsPerThread = BM * kChunksPerRow / kGemmThreads;  // 4

// chunk position of (row, chunk) inside a tile row: rows that share LDS banks get distinct
// positions both for 8 and for 16 consecutive rows read at one chunk index
__device__ __forceinline__ int swz(int row, int chunk)
{
    const int g = (((row >> 2) & 1) << 1) | (((row >> 1) ^ (row >> 3)) & 1);
    return chunk ^ g;
}

// order-preserving unsigned key of a float (and back): integer atomics then find extremes
__device__ __forceinline__ uint32_t ykey(float f)
{
    const uint32_t b = __float_as_uint(f);
    return (b & 0x80000000u) ? ~b : (b | 0x80000000u);
}
__device__ __forceinline__ float ykey_float(uint32_t k)
{
    return __uint_as_float((k & 0x80000000u) ? (k & 0x7fffffffu) : ~k);
}

__global__ __launch_bounds__(kGemmThreads) void gemm_i8_generic(GemmArgs g)
{
    extern __shared__ __attribute__((aligned(16))) char lds[];
    // [buffer][A | B][kTileBytes]
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = tid >> 6;
    const int wm = wave >> 1, wn = wave & 1;

    // ---- workgroup -> output tile.  Consecutive workgroup ids go round-robin over the XCDs,
    // so id % 8 names the XCD; each XCD walks its own sequence of patch_m x patch_n patches.
    const int b = blockIdx.x;
    const int xcd = b % kXcdCount;
    const int seq = b / kXcdCount;
    const int per_patch = g.patch_m * g.patch_n;
    const int patch = (seq / per_patch) * kXcdCount + xcd;
    if (patch >= g.n_patches) return;
    const int within = seq % per_patch;
    const int pm = patch / g.patches_n, pn = patch % g.patches_n;
    const int tile_m = pm * g.patch_m + within % g.patch_m;
    const int tile_n = pn * g.patch_n + within / g.patch_m;
    if (tile_m >= g.tiles_m || tile_n >= g.tiles_n) return;
    const int64_t m0 = (int64_t)tile_m * BM, n0 = (int64_t)tile_n * BN;

    // ---- global -> register staging: thread owns chunk (tid % 4) of rows tid/4 + 64 i
    const int ld_chunk = tid & (kChunksPerRow - 1);
    const int ld_row = tid / kChunksPerRow;
    const int8_t* a_ptr[kLoadsPerThread];
    const int8_t* b_ptr[kLoadsPerThread];
    int lds_off[kLoadsPerThread];
#pragma unroll
    for (int i = 0; i < kLoadsPerThread; ++i) {
        const int row = ld_row + i * (kGemmThreads / kChunksPerRow);
        // rows past the edge re-read the last valid row; their results are never stored
        const int64_t ra = min(m0 + row, g.T - 1), rb = min(n0 + row, g.N - 1);
        a_ptr[i] = g.A + ra * kPanel + ld_chunk * 16;
        b_ptr[i] = g.B + rb * kPanel + ld_chunk * 16;
        lds_off[i] = row * BK + swz(row, ld_chunk) * 16;
    }
    v4i ra[kLoadsPerThread], rb[kLoadsPerThread];
    const int nk = (int)panel_count(g.K);
    const int64_t panelA = g.T * kPanel, panelB = g.N * kPanel;

    auto load_global = [&](int kt) {
        // the last panel is zero filled past K in both operands
#pragma unroll
        for (int i = 0; i < kLoadsPerThread; ++i) {
            ra[i] = *reinterpret_cast<const v4i*>(a_ptr[i] + kt * panelA);
            rb[i] = *reinterpret_cast<const v4i*>(b_ptr[i] + kt * panelB);
        }
    };
    auto store_lds = [&](int buf) {
        char* base = lds + buf * 2 * kTileBytes;
#pragma unroll
        for (int i = 0; i < kLoadsPerThread; ++i) {
            *reinterpret_cast<v4i*>(base + lds_off[i]) = ra[i];
            *reinterpret_cast<v4i*>(base + kTileBytes + lds_off[i]) = rb[i];
        }
    };

    v16i acc[4][4];
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[i][j][v] = 0;

    // operand fragment addresses: lane reads row (lane % 32) of a 32-row sub-tile, 16-byte
    // chunk (lane / 32) + 2 kk of the tile row
    const int fr_row = lane & 31;
    const int fr_half = lane >> 5;

    load_global(0);
    store_lds(0);
    __syncthreads();

    for (int kt = 0; kt < nk; ++kt) {
        if (kt + 1 < nk) load_global(kt + 1);
        const char* a_base = lds + (kt & 1) * 2 * kTileBytes;
        const char* b_base = a_base + kTileBytes;
#pragma unroll
        for (int kk = 0; kk < BK / 32; ++kk) {
            v4i af[4], bf[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int row = wm * 128 + i * 32 + fr_row;
                af[i] = *reinterpret_cast<const v4i*>(a_base + row * BK + swz(row, kk * 2 + fr_half) * 16);
            }
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const int row = wn * 128 + j * 32 + fr_row;
                bf[j] = *reinterpret_cast<const v4i*>(b_base + row * BK + swz(row, kk * 2 + fr_half) * 16);
            }
#pragma unroll
            for (int i = 0; i < 4; ++i)
#pragma unroll
                for (int j = 0; j < 4; ++j)
                    acc[i][j] = __builtin_amdgcn_mfma_i32_32x32x32_i8(af[i], bf[j], acc[i][j], 0, 0, 0);
        }
        if (kt + 1 < nk) store_lds((kt + 1) & 1);
        __syncthreads();
    }

    // ---- epilogue.  Accumulator register v of lane l in sub-tile (i, j) is the element
    // row 8 (v / 4) + 4 (l / 32) + v % 4, column l % 32.
    const int64_t col_base = n0 + wn * 128 + (lane & 31);
    const int64_t row_base = m0 + wm * 128 + 4 * (lane >> 5);

    if (g.out_i32) {
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                const int64_t t = row_base + i * 32 + 8 * (v >> 2) + (v & 3);
                if (t < g.T) {
#pragma unroll
                    for (int j = 0; j < 4; ++j) {
                        const int64_t n = col_base + j * 32;
                        if (n < g.N) g.out_i32[t * g.ldo + n] = acc[i][j][v];
                    }
                }
            }
    }

    if (g.out_deq) {
        const int zx = *g.act_zero - 128;
        const double sx = (double)*g.act_step;
        const int Ki = (int)g.K;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int64_t n = col_base + j * 32;
            if (n >= g.N) continue;
            const int64_t pi = g.w_per_tensor ? 0 : n;
            const int zw = g.zero_w[pi] - 128;
            if (zw < -128 || zw > 127 || zx < -128 || zx > 127) raise_status(g.status, AWEQ_ST_ZEROPOINT);
            const double scale = sx * (double)g.step_w[pi];
            const double bs = g.bias ? (double)g.bias[n] : 0.0;
            // integer part in wrap-around 32-bit arithmetic: the final value fits (|.| <= 255^2 K)
            const unsigned cn = (unsigned)Ki * (unsigned)zx * (unsigned)zw - (unsigned)zx * (unsigned)g.rowsum_w[n];
#pragma unroll
            for (int i = 0; i < 4; ++i)
#pragma unroll
                for (int v = 0; v < 16; ++v) {
                    const int64_t t = row_base + i * 32 + 8 * (v >> 2) + (v & 3);
                    if (t >= g.T) continue;
                    const unsigned iv = (unsigned)acc[i][j][v] + cn - (unsigned)zw * (unsigned)g.rowsum_x[t];
                    const float y = (float)((double)(int)iv * scale + bs);
                    if (g.out_f16) reinterpret_cast<_Float16*>(g.out_deq)[t * g.ldo + n] = (_Float16)y;
                    else reinterpret_cast<float*>(g.out_deq)[t * g.ldo + n] = y;
                }
        }
    }

    if (g.colsum_acc) {
        // per-lane column partials over the wavefront's 128 rows; groups of four fit in int32
        __syncthreads();  // the k-loop's LDS tiles are dead: reuse for the cross-wavefront sum
        long long* red = reinterpret_cast<long long*>(lds);  // [BN]
        long long cs[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            long long s = 0;
#pragma unroll
            for (int i = 0; i < 4; ++i)
#pragma unroll
                for (int v4 = 0; v4 < 4; ++v4) {
                    int part = 0;
#pragma unroll
                    for (int v = 0; v < 4; ++v) {
                        const int64_t t = row_base + i * 32 + 8 * v4 + v;
                        part += (t < g.T) ? acc[i][j][v4 * 4 + v] : 0;
                    }
                    s += part;
                }
            s += partner<5>(s);  // lanes l and l + 32 hold the same column
            cs[j] = s;
        }
        if (wm == 1 && lane < 32) {
#pragma unroll
            for (int j = 0; j < 4; ++j) red[wn * 128 + j * 32 + lane] = cs[j];
        }
        __syncthreads();
        if (wm == 0 && lane < 32) {
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const int64_t n = col_base + j * 32;
                if (n < g.N)
                    atomicAdd(reinterpret_cast<unsigned long long*>(&g.colsum_acc[n]),
                              (unsigned long long)(cs[j] + red[wn * 128 + j * 32 + lane]));
            }
        }
    }
}


// ---------------------------------------------------------------------------- fast kernel
namespace fast {
constexpr int kThreads = 512;
// Tile of 64 MI tokens (MI = 4: 256, MI = 2: 128) x 256 channels.  One panel of both operands is a slot of the ring; the
// epilogue's slabs (8 KiB per wavefront) use the last slot and what is behind the ring, 160 KiB with it.
template <int MI>
struct Tile {
    static constexpr int kRows = 64 * MI;
    static constexpr int kHalfA = kRows * kPanel;                 // activation rows of a slot, then 16 KiB of weight rows
    static constexpr int kSlot = kHalfA + BN * kPanel;            // 32 KiB / 24 KiB
    static constexpr int kSlots = MI == 4 ? 4 : 5;
    static constexpr int kAhead = kSlots - 1;                     // panels requested ahead of the one being multiplied
    static constexpr int kLoads = MI / 2 + 2;                     // load instructions per wavefront and panel
    static constexpr int kSlabs = kAhead * kSlot;                 // 96 KiB
    static constexpr int kLds = kSlabs + 8 * 8192;                // 160 KiB
};

// chunk swizzle for 64-byte slot rows: the four rows r, r + 4, r + 8, r + 12 share LDS banks,
// so 16 consecutive rows read at one chunk index land on distinct banks
__device__ __forceinline__ int f4(int r) { return (r >> 2) & 3; }

// LDS-DMA load the compiler does not track (it would otherwise wait for every outstanding one
// before each LDS read): lane i's 16 bytes land at lds_addr + 16 i, lds_addr wave-uniform.
// The global address is a wave-uniform base (SGPR pair) plus a 32-bit per-lane offset.
__device__ __forceinline__ void dma16(const int8_t* sbase, uint32_t voff, uint32_t lds_addr)
{
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" ::"s"(lds_addr), "v"(voff), "s"(sbase) : "memory");
}
template <int N>
__device__ __forceinline__ void wait_vm()
{
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
}

#define SB() __builtin_amdgcn_sched_barrier(0)
#define MF(A_, B_, i, j) acc[i][j] = __builtin_amdgcn_mfma_i32_32x32x32_i8(B_[j], A_[i], acc[i][j], 0, 0, 0)

// DEQ: 0 none, 1 fp32, 2 fp16.  Persistent: the grid is one workgroup per compute unit
// (a multiple of 8), workgroup b takes the ids b, b + grid, b + 2 grid, ...; the first panels
// of its next tile are requested before the epilogue of the current one starts, so the loads
// fly while the results are stored.
// EPI (with DEQ == 2): bit 0 collects the column statistics of the binary16 output, bit 1 quantises
// it for the next layer; STORE = false keeps the output itself from being written.
// Args: GemmArgs, or GroupArgs for several weights.
template <int MI, bool I32, int DEQ, bool COLSUM, int EPI = 0, bool STORE = true, class Args = GemmArgs>
__global__ __launch_bounds__(kThreads) void gemm_i8_fast(Args g)
{
    using TL = Tile<MI>;
    constexpr bool kGroup = std::is_same<Args, GroupArgs>::value;
    // The epilogue's short forms.  Not with the accumulators among the outputs, which the general form stores as fast or faster (us, short ->
    // general: 3515 tokens 4468 x 2008 with sums 50.4 -> 48.5, 5000 x 2500 x 1000 with sums 31.3 -> 30.2, with binary16 output too 46.3 -> 44.2,
    // 4096 x 4096 x 4096 with sums 68.2 -> 67.6); the statistics epilogue, and the quantising one that also stores 256-token tiles, have no
    // registers left.
    constexpr bool kQuick = EPI == 0 ? !I32 : EPI == 2 && !(STORE && MI == 4);
    // passes of the general form in one piece: all of them where it is the only form; beside the short ones as many as cost no registers
    // (the next layer's codes with |Z| beyond 4096, 1 -> 4: 1024 tokens 16384 x 4096 85.3 -> 84.3, 2000 x 4096 x 1024 28.1 -> 27.7; 8 spill)
    constexpr int kUnroll = !kQuick ? 8 : EPI != 0 ? 4 : 1;
    constexpr bool kMayShare = kQuick && DEQ == 2 && EPI == 0 && !COLSUM && MI == 4;   // has the form for rows that share lines (kShared)
    constexpr int kSlot = TL::kSlot, kHalfA = TL::kHalfA, kAhead = TL::kAhead, kLoads = TL::kLoads;
    extern __shared__ __attribute__((aligned(1024))) char lds[];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave >> 2, wn = wave & 3;
    const int stride = gridDim.x;

    int vb = blockIdx.x, tile_m = 0, tile_n = 0;
    while (vb < g.n_ids && !tile_of(g, vb, tile_m, tile_n)) vb += stride;
    if (vb >= g.n_ids) return;

    const int64_t panelA = g.T * kPanel, panelB = g.N * kPanel;
    const int nh = (int)panel_count(g.K);
    const int pre = nh < kAhead ? nh : kAhead;
    const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char*)lds;
    const uint32_t wave_offA = wave * (512 * MI), wave_offB = kHalfA + wave * 2048;

    // global -> LDS: wave w brings tile rows 32 w .. 32 w + 31 of the weight and 8 MI w .. of the activations, 16 rows
    // x 64 B per instruction; lane i sits at row i / 4, chunk slot i % 4 and fetches chunk slot ^ f4(row)
    uint32_t oa[MI / 2], ob[2];  // byte offsets from the tile's first row inside a panel: < 16 KiB
    const int8_t* srcA;     // the tile's rows in the panel being fetched
    const int8_t* srcB;
    int64_t m0, n0;
    int member = 0;         // (kGroup) the weight of that tile

#define DMA_A(q) dma16(srcA, oa[q], dst_slot + wave_offA + (q) * 1024)
#define DMA_B(q) dma16(srcB, ob[q], dst_slot + wave_offB + (q) * 1024)
    // addresses of tile (tm, tn) and its first `pre` panels on their way into slots 0 ..
    auto start_tile = [&](int tm, int tn) {
        // (wave-uniform by construction; say so, the panel base addresses live in scalar registers)
        m0 = (int64_t)__builtin_amdgcn_readfirstlane(tm) * TL::kRows;
        if constexpr (kGroup) {
            member = __builtin_amdgcn_readfirstlane(tn / g.member_tiles);
            tn -= member * g.member_tiles;
        }
        n0 = (int64_t)__builtin_amdgcn_readfirstlane(tn) * BN;
        // rows past the edge re-read the last valid row; their results are never stored
        int lane_ = lane;
        asm volatile("" : "+v"(lane_));   // (hidden: formed again for every tile instead of living through the multiplications)
        const int last_m = (int)min((int64_t)TL::kRows, g.T - m0) - 1, last_n = (int)min((int64_t)BN, g.N - n0) - 1;
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            const int sub = q * 16 + (lane_ >> 2), chunk = (lane_ & 3) ^ f4(sub);   // (wavefronts start at multiples of 16 rows)
            if (q < MI / 2) oa[q] = (uint32_t)(min(wave * (8 * MI) + sub, last_m) * (int)kPanel + chunk * 16);
            ob[q] = (uint32_t)(min(wave * 32 + sub, last_n) * (int)kPanel + chunk * 16);
        }
        srcA = g.A + m0 * kPanel;
        if constexpr (kGroup) srcB = g.m[member].B + n0 * kPanel;
        else srcB = g.B + n0 * kPanel;
        for (int h = 0; h < pre; ++h) {
            const uint32_t dst_slot = lds0 + h * kSlot;
            DMA_A(0); DMA_B(0);
            if constexpr (MI == 4) DMA_A(1);
            DMA_B(1);
            srcA += panelA; srcB += panelB;
        }
    };

    start_tile(tile_m, tile_n);
    if (pre == kAhead) wait_vm<(kAhead - 1) * kLoads>(); else wait_vm<0>();

    // Vector memory operations of a wave complete in the order issued.  A tile that lies inside
    // the output issues at least kStores stores per wave after requesting the next tile's first
    // kAhead panels, so "at most kStores operations pending" means those panels have landed
    // while the stores may still be on their way (relaxed: set for the tile that follows).
    static_assert(EPI == 0 || DEQ == 2, "the fused epilogues work on the binary16 output");
    // MI sub-tile rows x 8 passes each, per kind of output; the atomics of the fused epilogues come
    // on top and are not counted: a lower bound is what the relaxed wait needs
    constexpr int kStoresAll = 8 * MI * ((I32 ? 1 : 0) + (DEQ != 0 && STORE ? 1 : 0) + ((EPI & 2) != 0 ? 1 : 0));
    constexpr int kStores = kStoresAll > 63 ? 63 : kStoresAll;
    bool relaxed = false;

    for (;;) {
        const int64_t cm0 = m0, cn0 = n0;   // the tile being multiplied
        const int cmember = member;
        v16i acc[MI][2];
#pragma unroll
        for (int i = 0; i < MI; ++i)
#pragma unroll
            for (int j = 0; j < 2; ++j)
#pragma unroll
                for (int v = 0; v < 16; ++v) acc[i][j][v] = 0;
        // fragment of K-step ks of a panel: lane reads row lane % 32 of a 32-row sub-tile, chunk
        // 2 ks + lane / 32 (sub-tiles start at multiples of 32 rows, so f4(row) = f4(lane % 32))
        // (formed again for every tile instead of living through the epilogue)
        int fl_ = lane;
        asm volatile("" : "+v"(fl_));
        const int fr_row = fl_ & 31, fr_half = fl_ >> 5;
        int offA[2], offB[2];
#pragma unroll
        for (int ks = 0; ks < 2; ++ks) {
            offA[ks] = (wm * (32 * MI) + fr_row) * kPanel + ((ks * 2 + fr_half) ^ f4(fr_row)) * 16;
            offB[ks] = kHalfA + (wn * 64 + fr_row) * kPanel + ((ks * 2 + fr_half) ^ f4(fr_row)) * 16;
        }
        v4i a0[MI], b0[2], a1[MI], b1[2];

#define RDA(dst, ks, i) dst[i] = *reinterpret_cast<const v4i*>(st + offA[ks] + (i) * 32 * kPanel)
#define RDB(dst, ks, j) dst[j] = *reinterpret_cast<const v4i*>(st + offB[ks] + (j) * 32 * kPanel)
        __builtin_amdgcn_s_barrier();  // panel 0 has landed for every wave
        {
            const char* st = lds;
#pragma unroll
            for (int i = 0; i < MI; ++i) RDA(a0, 0, i);
            RDB(b0, 0, 0); RDB(b0, 0, 1);
        }

        // one panel (64 bytes of K) = two K-steps of 2 MI MFMAs per wave.  F0 / F1 are the two
        // fragment register sets; each K-step multiplies one and fetches the other.  ISSUE: panel
        // h + kAhead is fetched into the slot panel h - 1 occupied (every wave finished reading it before
        // the barrier of panel h - 1).  WAITN: loads this wave may leave in flight when panel h + 1
        // has to be complete (kLoads per panel issued after it).
        uint32_t slot = 0;   // byte offset of panel h's slot
        auto half = [&](int h, auto issue_c, auto waitn_c, auto next_c) {
            constexpr bool ISSUE = decltype(issue_c)::value;
            constexpr int WAITN = decltype(waitn_c)::value;
            constexpr bool NEXT = decltype(next_c)::value;
            if constexpr (MI == 4) slot = (h & 3) * kSlot;
            const uint32_t next_slot = MI == 4 ? ((h + 1) & 3) * kSlot : slot == kAhead * kSlot ? 0 : slot + kSlot;
            const uint32_t dst_slot = lds0 + (MI == 4 ? ((h + 3) & 3) * kSlot : slot == 0 ? kAhead * kSlot : slot - kSlot);
            const char* st = lds + slot;
            SB();
            if constexpr (MI == 4) {
                RDA(a1, 1, 0); RDB(b1, 1, 0); RDB(b1, 1, 1); MF(a0, b0, 0, 0);
                SB();
                if constexpr (ISSUE) DMA_A(0);
                RDA(a1, 1, 1); RDA(a1, 1, 2); MF(a0, b0, 0, 1);
                SB();
                if constexpr (ISSUE) DMA_B(0);
                RDA(a1, 1, 3); MF(a0, b0, 1, 0);
                SB();
                if constexpr (ISSUE) DMA_A(1);
                MF(a0, b0, 1, 1);
                SB();
                if constexpr (ISSUE) DMA_B(1);
                MF(a0, b0, 2, 0); MF(a0, b0, 2, 1); MF(a0, b0, 3, 0); MF(a0, b0, 3, 1);
            } else {
                RDA(a1, 1, 0); RDB(b1, 1, 0); MF(a0, b0, 0, 0);
                SB();
                if constexpr (ISSUE) DMA_A(0);
                RDB(b1, 1, 1); RDA(a1, 1, 1); MF(a0, b0, 0, 1);
                SB();
                if constexpr (ISSUE) DMA_B(0);
                MF(a0, b0, 1, 0);
                SB();
                if constexpr (ISSUE) DMA_B(1);
                MF(a0, b0, 1, 1);
            }
            SB();
            if constexpr (ISSUE) { srcA += panelA; srcB += panelB; }
            if constexpr (NEXT) {
                // my loads of the next panel have landed, my reads of this one are done; after the
                // barrier that holds for every wave
                wait_vm<WAITN>();
                asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
                __builtin_amdgcn_s_barrier();
                SB();
                st = lds + next_slot;
                RDA(a0, 0, 0); RDB(b0, 0, 0); RDB(b0, 0, 1); MF(a1, b1, 0, 0);
                SB();
                if constexpr (MI == 4) {
                    RDA(a0, 0, 1); RDA(a0, 0, 2); MF(a1, b1, 0, 1);
                    SB();
                    RDA(a0, 0, 3); MF(a1, b1, 1, 0);
                    SB();
                    MF(a1, b1, 1, 1); MF(a1, b1, 2, 0); MF(a1, b1, 2, 1); MF(a1, b1, 3, 0); MF(a1, b1, 3, 1);
                } else {
                    RDA(a0, 0, 1); MF(a1, b1, 0, 1);
                    SB();
                    MF(a1, b1, 1, 0); MF(a1, b1, 1, 1);
                }
                SB();
            } else {
#pragma unroll
                for (int i = 0; i < MI; ++i) { MF(a1, b1, i, 0); MF(a1, b1, i, 1); }
            }
            if constexpr (MI != 4) slot = next_slot;
        };
        using std::integral_constant;
        int h = 0;
        if (relaxed) {
            // the panels requested before the epilogue landed together with panel 0: nothing to wait for, and a count
            // here would wait for the previous tile's stores
#pragma unroll
            for (; h < kAhead - 1; ++h) half(h, std::true_type{}, integral_constant<int, 63>{}, std::true_type{});
        }
        for (; h + kAhead < nh; ++h) half(h, std::true_type{}, integral_constant<int, (kAhead - 1) * kLoads>{}, std::true_type{});
        if constexpr (kAhead > 3) {
            if (h + 3 < nh) { half(h, std::false_type{}, integral_constant<int, 2 * kLoads>{}, std::true_type{}); ++h; }
        }
        if (h + 2 < nh) { half(h, std::false_type{}, integral_constant<int, kLoads>{}, std::true_type{}); ++h; }
        if (h + 1 < nh) { half(h, std::false_type{}, integral_constant<int, 0>{}, std::true_type{}); ++h; }
        half(h, std::false_type{}, integral_constant<int, 0>{}, std::false_type{});
#undef RDA
#undef RDB

        // ---- epilogue.  With the weight fragment as first MFMA operand, register v of lane l in
        // sub-tile (i, j) is token t = m0 + 32 MI wm + 32 i + l % 32 and output channel
        // n = n0 + 64 wn + 32 j + 8 (v / 4) + 4 (l / 32) + v % 4: four consecutive n per register quad.
        // Each wave turns its 32 (t) x 64 (n) slab of sub-tile row i around in a private 8 KiB LDS
        // region (rows of 256 bytes, 16-byte chunks XOR swizzled: conflict-free both ways) so that a
        // lane then holds 16 bytes of one output row and 16 lanes cover 256 contiguous bytes per store.
        // The slabs live in the last ring slot and behind the ring; the next tile's first kAhead
        // panels are already on their way into the other slots.
        // (hidden: what follows from the lane is formed here again for every tile instead of living through the multiplications)
        int lane_ = lane;
        asm volatile("" : "+v"(lane_));
        const int rd_r = lane_ >> 4, rd_c = lane_ & 15;
        const int64_t t_lane = cm0 + wm * (32 * MI) + rd_r;              // + 32 i + 4 p
        const int64_t n = cn0 + wn * 64 + rd_c * 4;                // this lane's four channels
        const bool n_ok = n < g.N;                                 // N % 4 == 0: all four or none

        const float* step_w;
        const int32_t *zero_w, *rowsum_w;
        const float* bias;
        void* out_deq;
        if constexpr (kGroup) {
            const GroupArgs::Member& o = g.m[cmember];
            step_w = o.step_w; zero_w = o.zero_w; rowsum_w = o.rowsum_w; bias = o.bias; out_deq = o.out_deq;
        } else {
            step_w = g.step_w; zero_w = g.zero_w; rowsum_w = g.rowsum_w; bias = g.bias; out_deq = g.out_deq;
        }
        // everything the epilogue reads from memory is requested before the next tile's panels,
        // so that waiting for it does not wait for them
        int rsx[MI / 2] = {};   // row sums of this wave's 32 MI tokens, one per lane and 64: token 64 h + lane
        Float4 sw = {{0.f, 0.f, 0.f, 0.f}}, bs = {{0.f, 0.f, 0.f, 0.f}};
        int nzw[4] = {0, 0, 0, 0};          // -Z'w = 128 - Z_w of this lane's channels
        unsigned cn[4] = {0, 0, 0, 0};      // K Z'x Z'w - Z'x rowsum_w, in wrap-around 32-bit arithmetic
        uint32_t est = 0;                   // status bits this lane raises for the tile
        int zx = 0;
        float sxf = 0.f;
        if constexpr (DEQ != 0) {
            zx = *g.act_zero - 128;
            sxf = *g.act_step;
            zx = __builtin_amdgcn_readfirstlane(zx);
            sxf = __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(sxf)));
            // the integer part is formed in 32-bit arithmetic: exact while it fits, which zero points in
            // [0, 255] guarantee for K <= 32768; anything else is flagged
            if (zx < -128 || zx > 127) est |= AWEQ_ST_ZEROPOINT;
#pragma unroll
            for (int hh = 0; hh < MI / 2; ++hh) {
                const int64_t t = cm0 + wm * (32 * MI) + hh * 64 + lane;
                rsx[hh] = t < g.T ? g.rowsum_x[t] : 0;
            }
            if (n_ok) {
                v4i zw4;
                if (g.w_per_tensor) {
                    const float s0 = step_w[0];
                    const int z0 = zero_w[0];
                    sw = Float4{{s0, s0, s0, s0}};
                    zw4 = v4i{z0, z0, z0, z0};
                } else {
                    sw = *reinterpret_cast<const Float4*>(step_w + n);
                    zw4 = *reinterpret_cast<const v4i*>(zero_w + n);
                }
                const v4i rw4 = *reinterpret_cast<const v4i*>(rowsum_w + n);
#pragma unroll
                for (int c = 0; c < 4; ++c) {
                    nzw[c] = 128 - zw4[c];
                    if (zw4[c] < 0 || zw4[c] > 255) est |= AWEQ_ST_ZEROPOINT;
                    cn[c] = 0u - (unsigned)g.K * (unsigned)zx * (unsigned)nzw[c] - (unsigned)zx * (unsigned)rw4[c];
                }
                if (bias) bs = *reinterpret_cast<const Float4*>(bias + n);
            }
            // pin the values in registers here: the compiler's wait for them then sits before the
            // panel requests below, which it cannot see, instead of behind them
#pragma unroll
            for (int hh = 0; hh < MI / 2; ++hh) asm volatile("" : "+v"(rsx[hh]));
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                asm volatile("" : "+v"(sw.f[c]));
                asm volatile("" : "+v"(bs.f[c]));
                asm volatile("" : "+v"(nzw[c]));
                asm volatile("" : "+v"(cn[c]));
            }
        }
        // Which form this tile's rows take (wave-uniform): kPlain, every row and channel inside; kShared, the same, with stores that stay in the
        // caches; kEdge, rows or channels past the edge; kGeneral, constants outside what the short arithmetic of the others covers.
        bool odd = false;   // this lane's channels have such constants
        Float4 nis = {{1.f, 1.f, 1.f, 1.f}};   // the next layer's 1 / s for this lane's four channels
        float nstep = 1.0f, nrstep = 1.0f, nthr = 0.0f;
        int nzero = 0;
        bool nscreen = false;
        if constexpr ((EPI & 2) != 0) {
            if (n_ok) nis = *reinterpret_cast<const Float4*>(g.next_inv_s + n);
            const ActParams np_ = quot_params(*g.next_step, *g.next_zero);
            nstep = np_.step; nzero = np_.zero; nrstep = np_.rstep; nthr = np_.thr;
            // the one-FMA quotient with its distance-to-tie test (see the activation quantizer): valid
            // for this lane if no binary16 value times its 1 / s can reach a quotient of 2^24
            nscreen = np_.screen;
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                asm volatile("" : "+v"(nis.f[c]));
                nscreen = nscreen && 65600.0f * fabsf(nis.f[c]) * nrstep < 16777216.0f;
                // (finite constants and 1 / s > 0: no quotient is a NaN, which the distance-to-tie test would not see)
                odd = odd || !(nis.f[c] > 0.0f && nis.f[c] < INFINITY) || !(fabsf(sxf * sw.f[c]) < INFINITY) || !(fabsf(bs.f[c]) < INFINITY);
            }
            odd = odd || !np_.screen;
            nstep = __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(nstep)));
            nrstep = __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(nrstep)));
            nthr = __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(nthr)));
            nzero = __builtin_amdgcn_readfirstlane(nzero);
        }

        // next tile of this workgroup
        int nvb = vb + stride, ntm = 0, ntn = 0;
        while (nvb < g.n_ids && !tile_of(g, nvb, ntm, ntn)) nvb += stride;
        const bool more = nvb < g.n_ids;
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        __builtin_amdgcn_s_barrier();  // every wave is done reading the ring
        if (more) start_tile(ntm, ntn);

        enum { kPlain, kShared, kEdge, kGeneral };
        int form = kGeneral;
        if constexpr (kQuick) {
            if constexpr (DEQ != 0) {
#pragma unroll
                for (int c = 0; c < 4; ++c) odd = odd || nzw[c] >= (1 << 23) || nzw[c] <= -(1 << 23);
            }
            const bool inside = cm0 + TL::kRows <= g.T && cn0 + BN <= g.N;
            // Rows that do not begin at multiples of 64 bytes share lines with the next tile's, written by another workgroup a little earlier
            // or later: non-temporal, halves of lines went to memory (us, binary16, non-temporal -> cached: 3515 tokens 4468 x 2008 38.1 -> 35.7,
            // 3900 x 4092 x 1024 24.6 -> 23.2, 8192 x 4092 x 1024 49.3 -> 43.8; but whole lines 4096 x 4096 x 1024 21.3 -> 24.3, with sums
            // over tokens 3900 x 4092 x 1024 28.3 -> 29.7, and where an eighth of the compute units have no tile less is written at a time:
            // 240 tiles 3800 x 4092 x 1024 / 4096 26.3 -> 25.4 / 61.9 -> 61.2, 208 tiles 3300 x 4092 23.2 -> 23.75 / 55.7 -> 55.9, 144 tiles
            // 2300 x 4092 19.1 -> 20.8 / 44.6 -> 46.0)
            const bool shared = kMayShare && ((reinterpret_cast<uintptr_t>(out_deq) | (uintptr_t)(g.ldo * 2)) & 63) != 0 &&
                                g.tiles_m * g.tiles_n > 224;
            if (__builtin_amdgcn_ballot_w64(odd && n_ok) == 0 && g.ldo < (1 << 28) && (!COLSUM || g.K < 32768))
                form = !inside ? kEdge : shared ? kShared : kPlain;
        }

        // per-channel constants of the de-quantisation
        double scale[4] = {0, 0, 0, 0}, bsd[4] = {0, 0, 0, 0};
        if constexpr (DEQ != 0) {
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                scale[c] = (double)sxf * (double)sw.f[c];
                bsd[c] = (double)bs.f[c];
            }
        }
        char* slab = lds + TL::kSlabs + wave * 8192;
        // The sums over tokens leave a wavefront as one atomic instruction of 64 neighbouring channels (lane 16 r + c: channel 4 c + r):
        // the memory side takes them by the line, and four instructions of every fourth channel cost more (binary16 output with
        // sums, 25003 tokens 768 x 768: 54.1 -> 38.9 us).
        // column sums of the accumulator itself (never of the corrected integer, which wraps for zero points far
        // outside [0, 255]: the sums the bias correction needs do not depend on zero points)
        long long csum[4] = {0, 0, 0, 0};
        int rows_in = 0;   // rows of this lane inside T (the fused code epilogue turns unsigned sums into signed ones)
        float ymn[4] = {INFINITY, INFINITY, INFINITY, INFINITY}, ymx[4] = {-INFINITY, -INFINITY, -INFINITY, -INFINITY};
        double ysum[4] = {0.0, 0.0, 0.0, 0.0};   // exact: at most 128 binary16 values each
        int rsy_kept[MI / 2] = {};               // row sums of the next layer's codes: one per lane and 64 tokens
        float cqf[4] = {0.f, 0.f, 0.f, 0.f};     // column sums of the next layer's unsigned codes over this tile (exact: 32 rows)
        const bool yq_pad = (EPI & 2) != 0 && !n_ok && cn0 + wn * 64 < g.N;   // zero fill of the last panel
        // the short forms: wave-uniform row pointers that move on by four tokens, the lane's offset from them, its tokens inside
        const int64_t wave_t = cm0 + wm * (32 * MI), wave_n = cn0 + wn * 64;
        char* row_deq = DEQ != 0 && STORE ? reinterpret_cast<char*>(out_deq) + (wave_t * g.ldo + wave_n) * (DEQ == 1 ? 4 : 2) : nullptr;
        char* row_yq = (EPI & 2) != 0 ? reinterpret_cast<char*>(g.yq) + ((wave_n >> 6) * g.T + wave_t) * kPanel : nullptr;
        const uint32_t lane_yq = (uint32_t)(rd_r * (int)kPanel + rd_c * 4);
        const uint32_t lane_elt = (uint32_t)rd_r * (uint32_t)g.ldo + (uint32_t)rd_c * 4;
        const int rows_t = (int)max((int64_t)0, min((int64_t)(32 * MI), g.T - t_lane)), lim = n_ok ? rows_t : 0;
        const _Float16 relu = g.act == 1 ? (_Float16)0.0f : (_Float16)__builtin_nanf("");   // max(y, NaN) = y
        const bool big_quot = __builtin_amdgcn_ballot_w64(!nscreen) != 0;
        const float qlim = nscreen ? INFINITY : 8388608.0f;          // (quotients up to 2^23: far outside the clamp, not yet flagged)
        int rsy_pairs = 0;       // code sums of two tokens (16 bits each): lane 16 r + u has the passes 2 u and 2 u + 1
        uint32_t cq02 = 0, cq13 = 0;   // column sums of the unsigned codes, two channels (16 bits each: 32 rows)
        int cpart[4] = {0, 0, 0, 0};
        // fp64 product and sum of the exact integer, as in the general form; |Z'w| and |row sum| < 2^23: a 24-bit multiply-add
        auto dequantise = [&](const v4i& o, int rs, float y[4]) {
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                const double div = (double)(int)((unsigned)o[c] + cn[c] + (unsigned)__mul24(nzw[c], rs));
                if constexpr (DEQ == 1) y[c] = (float)(div * scale[c] + bsd[c]);
                else y[c] = (float)__builtin_fma(div, scale[c], bsd[c]);
            }
        };
        typedef _Float16 h4 __attribute__((ext_vector_type(4)));
        typedef _Float16 h2 __attribute__((ext_vector_type(2)));
        auto rounded = [&](const float y[4], h2 oh[2]) {
            oh[0] = h2{(_Float16)y[0], (_Float16)y[1]};
            oh[1] = h2{(_Float16)y[2], (_Float16)y[3]};
            if constexpr ((EPI & 2) != 0) {
                const h2 lowest = {relu, relu};
                oh[0] = __builtin_elementwise_max(oh[0], lowest);
                oh[1] = __builtin_elementwise_max(oh[1], lowest);
            }
        };
        // the next layer's codes of four outputs by the one-FMA quotient, as unsigned bytes (the conversion clamps); tie: one of them is too
        // close to a tie for that
        auto next_codes = [&](const h2 oh[2], bool& tie) {
            const float zf = (float)nzero;
            float dmax = 0.0f, q[4];
            uint32_t w = 0;
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                q[c] = __builtin_fmaf(__builtin_fmaf((float)oh[c >> 1][c & 1], nis.f[c], 0.0f), nrstep, zf);
                const float n_ = rintf(q[c]);
                dmax = fmaxf(dmax, fabsf(q[c] - n_));
                w = __builtin_amdgcn_cvt_pk_u8_f32(n_, c, w);
            }
            if (big_quot) dmax = fmaxf(fmaxf(fabsf(q[0]), fabsf(q[1])), fmaxf(fabsf(q[2]), fabsf(q[3]))) > qlim ? 1.0f : dmax;
            tie = dmax > nthr;
            return w;
        };
        auto row_sum_of = [&](int i, int p) { return __builtin_amdgcn_ds_bpermute(((i & 1) * 32 + 4 * p) * 4 + rd_r * 4, rsx[i >> 1]); };
        auto slab_row = [&](int p) { return *reinterpret_cast<const v4i*>(slab + (4 * p + rd_r) * 256 + ((rd_c ^ (4 * (p & 3) + rd_r)) * 16)); };
        // The eight passes over sub-tile row i of the short forms.  A tile's epilogue is vector operations of 4.5 cycles each
        // with nothing multiplying meanwhile (the two wavefronts of a SIMD arrive together): 6 per output of a binary16 result, 14 with the
        // next layer's codes and the sums, where the general form takes 12 and 20 and waits for the LDS in every pass.  Shorter by: the
        // 24-bit multiply without its check, addresses that are a scalar and one offset, sums in 32 bits and in packed bytes, row sums two
        // tokens to a word, divisions for near ties afterwards.  (us, general form -> these: two layers 4096 -> 16384 -> 4096 of 4096
        // tokens 466 -> 449, three layers 4096 x 4096 of 8192 tokens inside their calibration 437 -> 418, the 128-token tiles of
        // 2048 tokens 4096 x 11008 89.3 -> 88.3.)
        auto short_rows = [&](int i, auto form_c) {
            constexpr bool EDGE = decltype(form_c)::value == kEdge, CACHED = decltype(form_c)::value == kShared;
            uint32_t redo = 0;
            int rsy_even = 0;
            // a pass's accumulators and row sum are requested one pass ahead
            v4i next_o = slab_row(0);
            int next_rs = DEQ != 0 ? row_sum_of(i, 0) : 0;
#pragma unroll 1
            for (int p4 = 0; p4 < 8; p4 += 4)
#pragma unroll
            for (int p_ = 0; p_ < 4; ++p_) {
                const int p = p4 + p_;
                const int pn = p_ < 3 ? p + 1 : (p4 + 4) & 7;   // (after the last one: the first again, not used)
                const v4i o = next_o;
                const int rs = next_rs;
                next_o = *reinterpret_cast<const v4i*>(slab + pn * 1024 + (rd_r * 256 + ((rd_c ^ (4 * ((p_ + 1) & 3) + rd_r)) * 16)));
                if constexpr (DEQ != 0) next_rs = row_sum_of(i, pn);
                SB();
                const bool in = !EDGE || i * 32 + 4 * p < lim;
                if constexpr (DEQ != 0) {
                    float y[4];
                    dequantise(o, rs, y);
                    if constexpr (DEQ == 1) {
                        typedef float f4 __attribute__((ext_vector_type(4)));
                        if (in) __builtin_nontemporal_store(f4{y[0], y[1], y[2], y[3]}, reinterpret_cast<f4*>(row_deq + (uint64_t)(lane_elt * 4u)));
                        row_deq += 16 * g.ldo;
                    } else {
                        h2 oh[2];
                        rounded(y, oh);
                        if constexpr (STORE) {
                            h4* const d = reinterpret_cast<h4*>(row_deq + (uint64_t)(lane_elt * 2u));
                            const h4 o4 = {oh[0][0], oh[0][1], oh[1][0], oh[1][1]};
                            if constexpr (CACHED) { if (in) *d = o4; }
                            else if (in) __builtin_nontemporal_store(o4, d);
                            row_deq += 8 * g.ldo;
                        }
                        if constexpr ((EPI & 2) != 0) {
                            bool tie;
                            uint32_t w = next_codes(oh, tie);
                            if constexpr (EDGE) { w = in ? w : 0u; tie = tie & in; }
                            redo |= __builtin_amdgcn_ballot_w64(tie) != 0 ? 1u << p : 0u;
                            cq02 += w & 0x00ff00ffu;
                            cq13 += (w >> 8) & 0x00ff00ffu;
                            w ^= 0x80808080u;   // u - 128 as a byte
                            if constexpr (EDGE) {
                                w = in ? w : 0u;
                                if (i * 32 + 4 * p < rows_t && (n_ok || yq_pad)) *reinterpret_cast<uint32_t*>(row_yq + (uint64_t)lane_yq) = w;
                            } else {
                                *reinterpret_cast<uint32_t*>(row_yq + (uint64_t)lane_yq) = w;
                            }
                            row_yq += 4 * kPanel;
                            // the 16 lanes of one output row, two passes at a time: 64 codes sum to 14 bits
                            const int d = __builtin_amdgcn_sdot4((int)w, 0x01010101, 0, false);
                            if ((p_ & 1) == 0) rsy_even = d;
                            else {
                                int both = (int)(((unsigned)d << 16) + (unsigned)rsy_even);
                                both += dpp_from<kXor1>(both);
                                both += dpp_from<kXor2>(both);
                                both += dpp_from<kRor4>(both);
                                both += dpp_from<kRor8>(both);
                                rsy_pairs = i * 4 + p / 2 == rd_c ? both : rsy_pairs;
                            }
                        }
                    }
                }
                if constexpr (COLSUM) {   // (eight accumulators fit 32 bits while K < 16384, four while K < 32768)
#pragma unroll
                    for (int c = 0; c < 4; ++c) {
                        cpart[c] += in ? o[c] : 0;
                        if (p_ == 3 && (p4 == 4 || g.K >= 16384)) { csum[c] += cpart[c]; cpart[c] = 0; }
                        else asm volatile("" : "+v"(cpart[c]));   // (summed here, not out of 32 kept values later)
                    }
                }
                SB();
            }
            if constexpr ((EPI & 2) != 0) {
                while (redo != 0) {   // (a wavefront's pass has such a code about once in 30)
                    const int p = __builtin_ctz(redo);
                    redo &= redo - 1;
                    const v4i o = slab_row(p);
                    float y[4];
                    h2 oh[2];
                    dequantise(o, row_sum_of(i, p), y);
                    rounded(y, oh);
                    bool tie;
                    const uint32_t w = next_codes(oh, tie);
                    if (tie && i * 32 + 4 * p < lim) {
                        uint32_t e = 0;
#pragma unroll
                        for (int c = 0; c < 4; ++c) e |= (uint32_t)quant_div((float)oh[c >> 1][c & 1] * nis.f[c], nstep, nzero, 255, est) << (8 * c);
                        cq02 += (e & 0x00ff00ffu) - (w & 0x00ff00ffu);
                        cq13 += ((e >> 8) & 0x00ff00ffu) - ((w >> 8) & 0x00ff00ffu);
                        *reinterpret_cast<uint32_t*>(row_yq - (8 - p) * (4 * kPanel) + (uint64_t)lane_yq) = e ^ 0x80808080u;
                        const int d = (int)__builtin_amdgcn_udot4(e, 0x01010101u, 0, false) - (int)__builtin_amdgcn_udot4(w, 0x01010101u, 0, false);
                        if (d != 0 && g.rowsum_y) atomicAdd(&g.rowsum_y[wave_t + i * 32 + 4 * p + rd_r], d);
                    }
                }
            }
        };
        auto turn = [&](int i) {
            int l_ = lane_;
            asm volatile("" : "+v"(l_));   // (eight addresses formed again for each sub-tile row rather than kept)
            const int wr_t = l_ & 31, wr_sw = wr_t & 15, wr_half = l_ >> 5;   // chunk (8 j + 2 q + l / 32) ^ (t & 15)
#pragma unroll
            for (int j = 0; j < 2; ++j)
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    v4i o = {acc[i][j][4 * q], acc[i][j][4 * q + 1], acc[i][j][4 * q + 2], acc[i][j][4 * q + 3]};
                    *reinterpret_cast<v4i*>(slab + wr_t * 256 + (((8 * j + 2 * q + wr_half) ^ wr_sw) * 16)) = o;
                }
        };
        if (kQuick && form == kPlain) {
#pragma unroll
            for (int i = 0; i < MI; ++i) { turn(i); short_rows(i, std::integral_constant<int, kPlain>{}); }
        } else if (kMayShare && form == kShared) {
#pragma unroll
            for (int i = 0; i < MI; ++i) { turn(i); short_rows(i, std::integral_constant<int, kShared>{}); }
        } else if (kQuick && form == kEdge) {
#pragma unroll
            for (int i = 0; i < MI; ++i) { turn(i); short_rows(i, std::integral_constant<int, kEdge>{}); }
        } else {
            int8_t* const yq_lane = (EPI & 2) != 0 ? g.yq + (((cn0 >> 6) + wn) * g.T) * kPanel + rd_c * 4 : nullptr;
#pragma unroll
            for (int i = 0; i < MI; ++i) {
                turn(i);
#pragma unroll kUnroll
                for (int p = 0; p < 8; ++p) {
                    const v4i o = slab_row(p);
                    const int64_t t = t_lane + i * 32 + 4 * p;
                    unsigned rs = 0;
                    int rsy = 0;   // this lane's share of the token's code sum for the next layer
                    // row sum of token 32 i + 4 p + lane / 16 of the wave: held by lane (that % 64), half
                    // i / 2 (fetched with every lane active: a switched-off source lane would read as 0)
                    if constexpr (DEQ != 0) rs = (unsigned)row_sum_of(i, p);
                    if (t < g.T && n_ok) {
                        if constexpr (I32) __builtin_nontemporal_store(o, reinterpret_cast<v4i*>(g.out_i32 + t * g.ldo + n));
                        if constexpr (DEQ != 0) {
                            float y[4];
#pragma unroll
                            for (int c = 0; c < 4; ++c) {
                                // |row sum| <= 128 K < 2^23 and |Z'w| < 2^23 for any zero point binary16 weights can
                                // produce: a 24-bit multiply (full rate); wider zero points take the 32-bit one
                                const unsigned zr = (nzw[c] < (1 << 23) && nzw[c] > -(1 << 23)) ? (unsigned)__mul24(nzw[c], (int)rs) : (unsigned)nzw[c] * rs;
                                const int iv = (int)((unsigned)o[c] + cn[c] + zr);
                                const double div = (double)iv;
                                // the binary32 output is the fp64 product and sum rounded once (two fp64 operations,
                                // like the definition); for binary16 one fused fp64 operation is far inside the rounding
                                // (the variant with both fused epilogues is out of registers: it widens the bias here)
                                const double bd = EPI == 3 ? (double)bs.f[c] : bsd[c];
                                if constexpr (DEQ == 1) y[c] = (float)(div * scale[c] + bd);
                                else y[c] = (float)__builtin_fma(div, scale[c], bd);
                            }
                            if constexpr ((EPI & 2) != 0) ++rows_in;
                            if constexpr (DEQ == 2) {
                                if constexpr (EPI != 0) {
                                    if (g.act == 1) {
#pragma unroll
                                        for (int c = 0; c < 4; ++c) y[c] = fmaxf(y[c], 0.0f);
                                    }
                                }
                                h4 oh = {(_Float16)y[0], (_Float16)y[1], (_Float16)y[2], (_Float16)y[3]};
                                if constexpr (STORE)
                                    __builtin_nontemporal_store(oh, reinterpret_cast<h4*>(reinterpret_cast<_Float16*>(out_deq) + t * g.ldo + n));
                                if constexpr ((EPI & 1) != 0) {
#pragma unroll
                                    for (int c = 0; c < 4; ++c) {
                                        const float yf = (float)oh[c];
                                        ymn[c] = fminf(ymn[c], yf);
                                        ymx[c] = fmaxf(ymx[c], yf);
                                        ysum[c] += (double)yf;
                                    }
                                }
                                if constexpr ((EPI & 2) != 0) {
                                    uint32_t w = 0;
                                    const float zf = (float)nzero;
                                    float cn_[4];
                                    float dmax = 0.0f;
#pragma unroll
                                    for (int c = 0; c < 4; ++c) {
                                        const float a = __builtin_fmaf((float)oh[c], nis.f[c], 0.0f);
                                        const float q = __builtin_fmaf(a, nrstep, zf);
                                        cn_[c] = rintf(q);
                                        dmax = fmaxf(dmax, fabsf(q - cn_[c]));
                                    }
                                    if (!nscreen || dmax > nthr) {
#pragma unroll
                                        for (int c = 0; c < 4; ++c)
                                            cn_[c] = (float)quant_div((float)oh[c] * nis.f[c], nstep, nzero, 255, est);
                                    }
#pragma unroll
                                    for (int c = 0; c < 4; ++c) {
                                        const float u = __builtin_amdgcn_fmed3f(cn_[c], 0.0f, 255.0f);
                                        cqf[c] += u;
                                        w = __builtin_amdgcn_cvt_pk_u8_f32(u, c, w);
                                    }
                                    w ^= 0x80808080u;   // u - 128 as a byte
                                    rsy = __builtin_amdgcn_sdot4((int)w, 0x01010101, 0, false);
                                    *reinterpret_cast<uint32_t*>(yq_lane + t * kPanel) = w;
                                }
                            } else {
                                typedef float f4 __attribute__((ext_vector_type(4)));
                                f4 of = {y[0], y[1], y[2], y[3]};
                                __builtin_nontemporal_store(of, reinterpret_cast<f4*>(reinterpret_cast<float*>(out_deq) + t * g.ldo + n));
                            }
                        }
                        if constexpr (COLSUM) {
#pragma unroll
                            for (int c = 0; c < 4; ++c) csum[c] += o[c];
                        }
                    } else if (yq_pad && t < g.T) {
                        *reinterpret_cast<uint32_t*>(yq_lane + t * kPanel) = 0u;
                    }
                    if constexpr ((EPI & 2) != 0) {
                        // the 16 lanes of one output row (every lane active here); lane 16 r + c keeps the sums of passes c and c + 16
                        rsy = group_allreduce<4>(rsy, OpAdd());
                        rsy_kept[i >> 1] = (i & 1) * 8 + p == rd_c ? rsy : rsy_kept[i >> 1];
                    }
                }
            }
        }
        if constexpr ((EPI & 1) != 0) {
            // lanes l, l ^ 16, l ^ 32 hold the same channels for different tokens
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                ymn[c] = fminf(ymn[c], partner<4>(ymn[c]));
                ymn[c] = fminf(ymn[c], partner<5>(ymn[c]));
                ymx[c] = fmaxf(ymx[c], partner<4>(ymx[c]));
                ymx[c] = fmaxf(ymx[c], partner<5>(ymx[c]));
                ysum[c] += partner<4>(ysum[c]);
                ysum[c] += partner<5>(ysum[c]);
            }
            if (n_ok && ymn[0] <= ymx[0]) {   // (no token of this tile row was inside T: nothing to add)
                const float lo = rd_r == 0 ? ymn[0] : rd_r == 1 ? ymn[1] : rd_r == 2 ? ymn[2] : ymn[3];
                const float hi = rd_r == 0 ? ymx[0] : rd_r == 1 ? ymx[1] : rd_r == 2 ? ymx[2] : ymx[3];
                atomicMin(&g.ykeys[n + rd_r], ykey(lo));
                atomicMax(&g.ykeys[g.N + n + rd_r], ykey(hi));
                // an integer: binary16 values are multiples of 2^-24
                double f = (rd_r == 0 ? ysum[0] : rd_r == 1 ? ysum[1] : rd_r == 2 ? ysum[2] : ysum[3]) * 16777216.0;
                if (!(fabs(f) < 9.0e18)) { f = 0.0; est |= AWEQ_ST_NONFINITE; }
                atomicAdd(reinterpret_cast<unsigned long long*>(&g.yfix[n + rd_r]), (unsigned long long)(long long)f);
            }
        }
        if constexpr ((EPI & 2) != 0) {
            if (form != kGeneral) {
                rows_in = (lim + 3) >> 2;
#pragma unroll
                for (int h = 0; h < MI / 2; ++h) {   // lane 16 r + c: pass 16 h + c
                    const int both = __builtin_amdgcn_ds_bpermute((rd_r * 16 + h * 8 + (rd_c >> 1)) * 4, rsy_pairs);
                    const int even = (int)(short)both;
                    rsy_kept[h] = (rd_c & 1) != 0 ? (both - even) >> 16 : even;
                }
            }
            // (one atomic instruction per 64 neighbouring tokens; four tokens at a time, the two layers 4096 -> 16384 -> 4096 took
            // 172 instead of 157 us at 1024 tokens, 110 instead of 100 at 512)
            if (g.rowsum_y) {
#pragma unroll
                for (int h = 0; h < MI / 2; ++h) {
                    const int64_t t = t_lane + h * 64 + rd_c * 4;   // pass c of 16: token 32 (c / 8) + 4 (c % 8) + r = 4 c + r
                    if (t < g.T) atomicAdd(&g.rowsum_y[t], rsy_kept[h]);
                }
            }
            int cq[4];
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                cq[c] = (form != kGeneral ? (int)((((c & 1) ? cq13 : cq02) >> (8 * (c & 2))) & 0xffffu) : (int)cqf[c]) - 128 * rows_in;
                cq[c] += partner<4>(cq[c]);
                cq[c] += partner<5>(cq[c]);
            }
            const int v = rd_r == 0 ? cq[0] : rd_r == 1 ? cq[1] : rd_r == 2 ? cq[2] : cq[3];
            if (n_ok && g.colsum_yq) atomicAdd(reinterpret_cast<unsigned long long*>(&g.colsum_yq[n + rd_r]), (unsigned long long)(long long)v);
        }
        if constexpr (EPI != 0 || DEQ != 0) raise_status(g.status, est);
        if constexpr (COLSUM) {
            // lanes l, l ^ 16, l ^ 32 hold the same channels for different tokens
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                csum[c] += partner<4>(csum[c]);
                csum[c] += partner<5>(csum[c]);
            }
            const long long v = rd_r == 0 ? csum[0] : rd_r == 1 ? csum[1] : rd_r == 2 ? csum[2] : csum[3];
            if (n_ok) atomicAdd(reinterpret_cast<unsigned long long*>(&g.colsum_acc[n + rd_r]), (unsigned long long)v);
        }
        if (!more) break;
        vb = nvb;
        // the panels requested before the epilogue have landed
        relaxed = kStores > 0 && nh >= 2 * kAhead && cm0 + TL::kRows <= g.T && cn0 + BN <= g.N;
        if (relaxed) wait_vm<kStores>();
        else wait_vm<0>();
    }
#undef DMA_A
#undef DMA_B
}
#undef SB
#undef MF
}  // namespace fast

__global__ void zero_fill_u32_gemm(uint32_t* p, int64_t n)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = 0u;
}


}  // namespace aweq

using namespace aweq;

namespace aweq {

// The tiled kernel's plan: tiles of 256 tokens, or of 128 (`half`) where their rounds of workgroups, each kHalfTileCost of
// a round of the larger ones, take less: a round lasts as long however few of the 256 compute units have a tile.
// (us, 256 -> 128 tokens per tile, binary16 output: 2048 tokens 4096 x 11008 147 -> 83.9, 4096 x 4096 63.0 -> 36.3; 1000 tokens 4096 x 4096 46.2 -> 34.8.)
static int plan_tiled(GemmArgs& g, bool& half, double& cost, int64_t& blocks)
{
    GemmArgs h = g;
    int64_t blocks_h = 0;
    const int rc = plan_walk(g, g.T, g.N, g.K, BM, blocks);
    if (rc != AWEQ_OK) return rc;
    cost = (double)rounds_of(g);
    // (from seven rounds on a workgroup's idle ids in some rounds make up for each other, which the count of rounds does not see: 8230 tokens
    // 14720 x 1024 / 14720 x 4096 169 / 487 with 256 tokens per tile, 176 / 501 with 128, modelled 9 and 8.55 rounds)
    half = plan_walk(h, h.T, h.N, h.K, BM / 2, blocks_h) == AWEQ_OK && kHalfTileCost * (double)rounds_of(h) < cost &&
           cdiv(g.T, BM) * cdiv(g.N, BM) <= 6 * 256;
    if (half) { g = h; cost = kHalfTileCost * (double)rounds_of(h); }
    return AWEQ_OK;
}

// Launches of their own leave compute units without a tile in each one's last round, and each has its launch, its ramp and its last epilogue, which do
// not grow with K: kTiledFixed us (the kernel for some hundred tokens the same; the few-token one kFewFixed, the read of its tokens, and per round of tile
// FewPlan::tile kFewShare of what it is modelled to take).
// (us, whole calibrations, a launch each -> one: three weights 4096 x 4096 of 512 tokens 135 -> 112, 2048 tokens 193 -> 186, 4096 tokens 274 -> 265, 2048 x
// 2048 of 700 tokens 77.8 -> 59.2, two 1024 x 1024 of 2048 tokens 46.8 -> 39.3, four 1024 x 4096 of 1024 tokens 88.8 -> 71.8; against it two
// 1024 x 1024 of 128 tokens 31.0 -> 35.2, two 512 x 512 of 512 tokens 27.1 -> 30.2, three 3072 x 3072 of 16 tokens 70.9 -> 77.3, four 1024 x 8192 of 16
// tokens 90.6 -> 106.)
// One launch of few panels takes kTiledLeast (two weights of up to 104 values a row: 36 x 104 of 408 tokens 25.5 -> 27.4, 976 x 80 of 10 tokens 25.2 -> 27.0,
// but three 28.0 -> 26.8).
constexpr double kTiledFixed = 3.0, kTiledLeast = 4.2, kFewFixed = 1.7, kFewToken = 0.25e-6;
constexpr double kFewShare[] = {0.75, 1.0, 0.88, 0.96, 0.92, 0.96};
int launch_gemm_i8_group(GroupArgs& g, int n, hipStream_t st)
{
    const int64_t N = g.N;
    g.member_tiles = (int)cdiv(N, BN);
    bool half = false, half_one = false;
    double cost = 0.0, one = 0.0;
    int64_t blocks = 0;
    GemmArgs a = g;
    int rc = plan_tiled(a, half_one, one, blocks);
    if (rc != AWEQ_OK) return rc;
    g.N = (int64_t)n * g.member_tiles * BN;
    rc = plan_tiled(g, half, cost, blocks);
    g.N = N;
    if (rc != AWEQ_OK) return rc;
    if (one > 8.0) return AWEQ_ERR_SHAPE;   // (many rounds: 32768 tokens 5952 x 5952 1901 -> 1908, 16384 tokens 8192 x 8192 the same)
    // what aweq_w8a8_gemm takes for each weight
    const double us = (double)g.K / 8192.0, tiled = kTiledRoundCost * one;
    const FewPlan few = plan_few(g.T, N);
    MidPlan mid = plan_mid(g.T, N);
    if (g.K <= 512 && mid.cost > 43.0) mid.cost *= 1.2;
    const bool by_few = few.cost <= mid.cost && few.cost < tiled, by_tiles = !by_few && mid.cost >= tiled;
    const double each = by_few ? kFewFixed + (double)(g.T * g.K) * kFewToken + kFewShare[few.tile] * few.cost * us
                               : kTiledFixed + (by_tiles ? tiled : mid.cost) * us;
    const double together = kTiledFixed + kTiledRoundCost * cost * us;
    if ((together > kTiledLeast ? together : kTiledLeast) > n * each) return AWEQ_ERR_SHAPE;
    // In as many rounds as launches of their own take.  One of 256-token tiles a weight that leaves compute units idle runs at a higher clock than the
    // full rounds of one launch, which loses the more the longer the rows and the fewer the tiles (two weights 4276 x 8624 of 2890 tokens, 204 tiles,
    // 347 -> 367, 2048 x 4096 of 6274, 200, 159 -> 168, but 3796 x 3144 of 3385, 210, 158 -> 153, and full rounds 2048 x 2048 of 4096 tokens 110 -> 105);
    // of 128-token tiles with rows much longer than the outputs (three 2048 x 11008 of 3000 tokens 347 -> 370, 1024 x 8192 of 6000 250 -> 266); and
    // weights that do not fit the memory-side cache together (four 8192 x 8192 of 2654 tokens 990 -> 1019, 6432 x 10344 of 1955 847 -> 932).  Over
    // 1750 groups without regard to these the launch each was faster by more than 1.5 % in 117, now in 11, by 4 % at most.
    if (by_tiles && cost > 0.94 * n * one) {
        const double idle = 1.0 - (double)a.tiles_m * a.tiles_n / (256.0 * (double)cdiv((int64_t)a.tiles_m * a.tiles_n, 256));
        if (!half_one && one <= 1.0 && (double)g.K * (idle - 0.05) > 300.0) return AWEQ_ERR_SHAPE;
        if (half_one && idle > 0.1 && g.K >= 4 * N) return AWEQ_ERR_SHAPE;
        if (n * N * g.K >= kCacheBytes) return AWEQ_ERR_SHAPE;
    }
    const void* fn = half ? reinterpret_cast<const void*>(fast::gemm_i8_fast<2, false, 2, false, 0, true, GroupArgs>)
                          : reinterpret_cast<const void*>(fast::gemm_i8_fast<4, false, 2, false, 0, true, GroupArgs>);
    return launch_persistent(fn, fast::kThreads, half ? fast::Tile<2>::kLds : fast::Tile<4>::kLds, &g, g.n_ids, st);
}

static void clear_fused(GemmArgs& g)
{
    g.w_per_tensor = 0;
    g.act = 0; g.ykeys = nullptr; g.yfix = nullptr; g.next_inv_s = nullptr; g.next_step = nullptr; g.next_zero = nullptr;
    g.yq = nullptr; g.rowsum_y = nullptr; g.colsum_yq = nullptr; g.status = nullptr;
}

// accumulators of the fused epilogues start from their identities (a fill kernel: graph-capturable)
__global__ void fused_init(long long* colsum_acc, uint32_t* ykeys, long long* yfix, int64_t N, long long* colsum_yq, int32_t* rowsum_y, int64_t T)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < N) {
        colsum_acc[i] = 0;
        if (ykeys) { ykeys[i] = 0xffffffffu; ykeys[N + i] = 0u; yfix[i] = 0; }
        if (colsum_yq) colsum_yq[i] = 0;
    }
    if (rowsum_y && i < T) rowsum_y[i] = 0;
}

// keys / fixed-point sums -> the outputs aweq_calib_stats would give on the stored output
__global__ void fused_stats_finish(const uint32_t* ykeys, const long long* yfix, int64_t N, int64_t T, float* cmin, float* cmax,
                                   double* csum, uint64_t* count, int accumulate, uint32_t* status)
{
    const int64_t n = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (n == 0 && count) *count = (accumulate ? *count : 0) + (uint64_t)T;
    if (n >= N) return;
    float a = ykey_float(ykeys[n]), b = ykey_float(ykeys[N + n]);
    double s = (double)yfix[n] * 5.9604644775390625e-08;   // 2^-24
    if (isinf(a) || isinf(b)) raise_status(status, AWEQ_ST_NONFINITE);
    if (accumulate) {
        a = fminf(a, cmin[n]);
        b = fmaxf(b, cmax[n]);
        if (csum) s += csum[n];
    }
    cmin[n] = a;
    cmax[n] = b;
    if (csum) csum[n] = s;
}

}  // namespace aweq

using namespace aweq;

extern "C" int aweq_w8a8_gemm(const void* X, aweq_dtype x_dt, int64_t T, int64_t K, int64_t ldx,
                              const float* inv_s, const float* act_step, const int32_t* act_zero,
                              int8_t* xq, int32_t* rowsum_x, int64_t* colsum_xq,
                              const int8_t* wq, int64_t N, const float* step_w, const int32_t* zero_w, int w_group,
                              const int32_t* rowsum_w, const float* bias,
                              int32_t* out_i32, void* out_deq, aweq_dtype out_dt, int64_t ldo,
                              int64_t* colsum_acc, void* ws, size_t ws_bytes,
                              uint32_t* status, void* stream)
{
    if (!X || !wq) return AWEQ_ERR_NULL;
    if (w_group != 0 && w_group != -1) return AWEQ_ERR_GROUP;
    if (x_dt != AWEQ_F32 && x_dt != AWEQ_F16 && x_dt != AWEQ_I8) return AWEQ_ERR_DTYPE;
    if (T <= 0 || N <= 0 || K <= 0 || (K % 8) != 0) return AWEQ_ERR_SHAPE;
    if (K > 32768) return AWEQ_ERR_SHAPE;  // keeps 128*128*K and 255*255*K inside int32
    const int8_t* a = nullptr;
    if (x_dt == AWEQ_I8) {
        if (ldx != K) return AWEQ_ERR_SHAPE;
        a = reinterpret_cast<const int8_t*>(X);
    } else {
        int rc = check_quant_act_args(X, x_dt, T, K, ldx, inv_s, act_step, act_zero, xq, false);
        if (rc != AWEQ_OK) return rc;
        rc = check_quant_act_ws(T, K, rowsum_x, colsum_xq, ws, ws_bytes);
        if (rc != AWEQ_OK) return rc;
        a = xq;
    }
    if (!aligned16(a) || !aligned16(wq)) return AWEQ_ERR_ALIGN;
    if (out_i32 || out_deq) {
        if (ldo < N) return AWEQ_ERR_SHAPE;
    }
    if (out_deq) {
        if (out_dt != AWEQ_F32 && out_dt != AWEQ_F16) return AWEQ_ERR_DTYPE;
        if (!act_step || !act_zero || !step_w || !zero_w || !rowsum_x || !rowsum_w) return AWEQ_ERR_NULL;
    }
    hipStream_t st = as_stream(stream);
    auto quantise = [&]() {
        return x_dt == AWEQ_I8 ? (int)AWEQ_OK : launch_quant_act(X, x_dt, T, K, ldx, inv_s, act_step, act_zero, xq, rowsum_x, colsum_xq, ws, status, st);
    };
    if (!out_i32 && !out_deq && !colsum_acc) {
        const int rc = quantise();
        return rc != AWEQ_OK ? rc : launch_status();
    }

    GemmArgs g;
    g.A = a; g.B = wq; g.T = T; g.N = N; g.K = K;
    g.out_i32 = out_i32; g.out_deq = out_deq; g.out_f16 = out_dt == AWEQ_F16; g.ldo = ldo;
    g.colsum_acc = reinterpret_cast<long long*>(colsum_acc);
    g.act_step = act_step; g.act_zero = act_zero; g.step_w = step_w; g.zero_w = zero_w;
    g.rowsum_x = rowsum_x; g.rowsum_w = rowsum_w; g.bias = bias;
    clear_fused(g);
    g.w_per_tensor = w_group == -1;
    g.status = status;
    // the fast kernel stores 16-byte output quads
    bool fast_ok = (N % 4) == 0;
    if (out_i32 && (!aligned16(out_i32) || (ldo % 4) != 0)) fast_ok = false;
    if (out_deq && (!aligned16(out_deq) || (ldo % 4) != 0 || (w_group == 0 && (!aligned16(step_w) || !aligned16(zero_w))) ||
                    !aligned16(rowsum_w) || (bias && !aligned16(bias))))
        fast_ok = false;
    // Up to 256 tokens and 256 channels are one 256 x 256 tile, whose workgroup has read everything before it stores: an output over an
    // input stays there (tiled_cost 0: no other form is cheaper).  The other forms would have several workgroups, one storing while another reads.
    const int64_t scales = g.w_per_tensor ? 4 : N * 4;
    const bool apart = !overlap({matrix_span(out_i32, T, N, ldo, 4), matrix_span(out_deq, T, N, ldo, dtype_size(out_dt))},
                                {{a, T * panel_count(K) * kPanel}, {wq, N * panel_count(K) * kPanel}, {rowsum_x, T * 4}, {rowsum_w, N * 4},
                                 {act_step, 4}, {act_zero, 4}, {step_w, scales}, {zero_w, scales}, {bias, N * 4}});
    bool half = false;
    double tiled_cost = 0.0;
    int64_t blocks = 0;
    const int prc = fast_ok && apart ? plan_tiled(g, half, tiled_cost, blocks) : plan_walk(g, g.T, g.N, g.K, BM, blocks);
    if (prc != AWEQ_OK) return prc;

    // the form whose rounds of workgroups are modelled to take least
    const FewPlan few = plan_few(T, N);
    MidPlan mid = plan_mid(T, N);
    // Short rows in several rounds are mostly epilogue, which the persistent tiled form overlaps with the next tile (us, 128 x 128 tiles / tiled:
    // 8583 tokens 1920 x 360 34.6 / 24.9, the GEMM of 2987 tokens 2688 x 160 18.2 / 17.0)
    if (K <= 512 && mid.cost > 43.0) mid.cost *= 1.2;
    // one to four tokens: the few-token form quantises them itself, one launch instead of two (us per call, one / four tokens:
    // 4096 x 4096 9.2 -> 7.9 / 9.4 -> 9.3, 11008 x 4096 14.8 -> 12.5 / 15.2 -> 14.2, 1536 x 2048 8.5 -> 6.0 / 8.5 -> 7.0; no more than
    // 16 KiB of codes: every workgroup repeats the work).  Not where an output lies over what the quantizer reads: a workgroup would
    // store it while another still reads; the quantizer's own launch is over before the GEMM stores anything.
    const bool own_quant = fast_ok && x_dt != AWEQ_I8 && !colsum_xq && T <= kQuantTokens && T * panel_count(K) * kPanel <= kQuantFewBytes && aligned16(inv_s) &&
                           few.cost <= mid.cost && few.cost < kTiledRoundCost * tiled_cost &&
                           !overlap({matrix_span(out_i32, T, N, ldo, 4), matrix_span(out_deq, T, N, ldo, dtype_size(out_dt)), {colsum_acc, N * 8}, {rowsum_x, T * 4}, {xq, T * panel_count(K) * kPanel}},
                                    {matrix_span(X, T, K, ldx, dtype_size(x_dt)), {inv_s, K * 4}, {act_step, 4}, {act_zero, 4}});
    if (!own_quant) {
        const int rc = quantise();
        if (rc != AWEQ_OK) return rc;
    }
    if (colsum_acc) zero_fill_u32_gemm<<<(unsigned)cdiv(2 * N, 256), 256, 0, st>>>(reinterpret_cast<uint32_t*>(colsum_acc), 2 * N);
    if (own_quant) return launch_gemm_i8_few_quant(g, few, QuantIn{X, ldx, inv_s, xq, rowsum_x}, x_dt == AWEQ_F16, st);
    if (fast_ok && few.cost <= mid.cost && few.cost < kTiledRoundCost * tiled_cost) return launch_gemm_i8_few(g, few, st);
    if (fast_ok && mid.cost < kTiledRoundCost * tiled_cost) return launch_gemm_i8_mid(g, mid, st);
    if (fast_ok) {
        const int deq = out_deq ? (out_dt == AWEQ_F16 ? 2 : 1) : 0;
        const void* fn = nullptr;
#define AWEQ_PICK(I, D, C)                                                                                             \
    if ((out_i32 != nullptr) == I && deq == D && (colsum_acc != nullptr) == C)                                         \
        fn = half ? reinterpret_cast<const void*>(fast::gemm_i8_fast<2, I, D, C>) : reinterpret_cast<const void*>(fast::gemm_i8_fast<4, I, D, C>);
        AWEQ_PICK(true, 0, true) AWEQ_PICK(true, 0, false) AWEQ_PICK(false, 0, true)
        AWEQ_PICK(true, 1, true) AWEQ_PICK(true, 1, false) AWEQ_PICK(false, 1, true) AWEQ_PICK(false, 1, false)
        AWEQ_PICK(true, 2, true) AWEQ_PICK(true, 2, false) AWEQ_PICK(false, 2, true) AWEQ_PICK(false, 2, false)
#undef AWEQ_PICK
        return launch_persistent(fn, fast::kThreads, half ? fast::Tile<2>::kLds : fast::Tile<4>::kLds, &g, g.n_ids, st);
    }
    const size_t lds_bytes = 2 * 2 * kTileBytes;  // 64 KiB
    int dev = 0, cus = 0;
    if (device_cus(dev, cus) != AWEQ_OK || raise_lds_limit(reinterpret_cast<const void*>(gemm_i8_generic), dev, (int)lds_bytes) != AWEQ_OK)
        return AWEQ_ERR_LAUNCH;
    gemm_i8_generic<<<(unsigned)blocks, kGemmThreads, lds_bytes, st>>>(g);
    return launch_status();
}

extern "C" int aweq_w8a8_gemm_fused(const int8_t* xq, int64_t T, int64_t K, const int8_t* wq, int64_t N,
                                    const float* act_step, const int32_t* act_zero,
                                    const float* step_w, const int32_t* zero_w,
                                    const int32_t* rowsum_x, const int32_t* rowsum_w, const float* bias, int act,
                                    void* out_f16, int64_t ldo, int64_t* colsum_acc,
                                    float* ycmin, float* ycmax, double* ycsum, uint64_t* ycount, int accumulate,
                                    const float* next_inv_s, const float* next_step, const int32_t* next_zero,
                                    int8_t* yq, int32_t* rowsum_y, int64_t* colsum_yq,
                                    void* ws, size_t ws_bytes, uint32_t* status, void* stream)
{
    if (!xq || !wq || !act_step || !act_zero || !step_w || !zero_w || !rowsum_x || !rowsum_w || !colsum_acc) return AWEQ_ERR_NULL;
    const bool want_stats = ycmin != nullptr, want_quant = yq != nullptr;
    if (!want_stats && !want_quant) return AWEQ_ERR_NULL;
    if (want_stats && !ycmax) return AWEQ_ERR_NULL;
    if (want_quant && (!next_inv_s || !next_step || !next_zero)) return AWEQ_ERR_NULL;
    if (act != 0 && act != 1) return AWEQ_ERR_SHAPE;
    if (T <= 0 || N <= 0 || K <= 0 || (K % 8) != 0 || K > 32768 || (N % 4) != 0) return AWEQ_ERR_SHAPE;
    if (out_f16 && (ldo < N || (ldo % 4) != 0)) return AWEQ_ERR_SHAPE;
    if (!aligned16(xq) || !aligned16(wq) || !aligned16(step_w) || !aligned16(zero_w) || !aligned16(rowsum_w) ||
        (bias && !aligned16(bias)) || (out_f16 && !aligned16(out_f16)) || (want_quant && (!aligned16(next_inv_s) || !aligned16(yq))))
        return AWEQ_ERR_ALIGN;
    if (want_stats && (!ws || ws_bytes < (size_t)N * 16)) return AWEQ_ERR_WORKSPACE;
    if (want_stats && !aligned16(ws)) return AWEQ_ERR_ALIGN;

    GemmArgs g;
    g.A = xq; g.B = wq; g.T = T; g.N = N; g.K = K;
    g.out_i32 = nullptr; g.out_deq = out_f16; g.out_f16 = 1; g.ldo = ldo;
    g.colsum_acc = reinterpret_cast<long long*>(colsum_acc);
    g.act_step = act_step; g.act_zero = act_zero; g.step_w = step_w; g.zero_w = zero_w;
    g.rowsum_x = rowsum_x; g.rowsum_w = rowsum_w; g.bias = bias;
    clear_fused(g);
    g.act = act; g.status = status;
    if (want_stats) {
        g.yfix = reinterpret_cast<long long*>(ws);
        g.ykeys = reinterpret_cast<uint32_t*>(g.yfix + N);
    }
    if (want_quant) {
        g.next_inv_s = next_inv_s; g.next_step = next_step; g.next_zero = next_zero;
        g.yq = yq; g.rowsum_y = rowsum_y; g.colsum_yq = reinterpret_cast<long long*>(colsum_yq);
    }
    const bool apart = !overlap({matrix_span(out_f16, T, N, ldo, 2), {yq, T * panel_count(N) * kPanel}},
                                {{xq, T * panel_count(K) * kPanel}, {wq, N * panel_count(K) * kPanel}, {rowsum_x, T * 4}, {rowsum_w, N * 4},
                                 {act_step, 4}, {act_zero, 4}, {step_w, N * 4}, {zero_w, N * 4}, {bias, N * 4},
                                 {next_inv_s, N * 4}, {next_step, 4}, {next_zero, 4}});   // (as in aweq_w8a8_gemm)
    bool half = false;
    double tiled_cost = 0.0;
    int64_t blocks = 0;
    const int prc = apart ? plan_tiled(g, half, tiled_cost, blocks) : plan_walk(g, g.T, g.N, g.K, BM, blocks);
    if (prc != AWEQ_OK) return prc;

    hipStream_t st = as_stream(stream);
    const int64_t init_n = (want_quant && rowsum_y && T > N) ? T : N;
    fused_init<<<(unsigned)cdiv(init_n, 256), 256, 0, st>>>(g.colsum_acc, g.ykeys, g.yfix, N, want_quant ? g.colsum_yq : nullptr,
                                                            want_quant ? rowsum_y : nullptr, T);
    // fewer tokens: 64 x 128 or 128 x 128 tiles, which have the quantising epilogue but not the statistics one (two layers
    // 4096 -> 16384 -> 4096, us, 128 tokens a tile -> these: 16 tokens 55.9 -> 47.3, 64 tokens 73.6 -> 62.3, 256 tokens 93.0 -> 83.7)
    const MidPlan mid = plan_mid(T, N);
    if (!want_stats && mid.cost < kTiledRoundCost * tiled_cost) return launch_gemm_i8_mid(g, mid, st);
    const int epi = (want_stats ? 1 : 0) | (want_quant ? 2 : 0);
    const bool store = out_f16 != nullptr;
    const void* fn = nullptr;
#define AWEQ_PICK(E, S)                                                                                                \
    if (epi == E && store == S)                                                                                        \
        fn = half ? reinterpret_cast<const void*>(fast::gemm_i8_fast<2, false, 2, true, E, S>)                         \
                  : reinterpret_cast<const void*>(fast::gemm_i8_fast<4, false, 2, true, E, S>);
    AWEQ_PICK(1, true) AWEQ_PICK(1, false) AWEQ_PICK(2, true) AWEQ_PICK(2, false) AWEQ_PICK(3, true) AWEQ_PICK(3, false)
#undef AWEQ_PICK
    const int rc = launch_persistent(fn, fast::kThreads, half ? fast::Tile<2>::kLds : fast::Tile<4>::kLds, &g, g.n_ids, st);
    if (rc != AWEQ_OK) return rc;
    if (want_stats)
        fused_stats_finish<<<(unsigned)cdiv(N, 256), 256, 0, st>>>(g.ykeys, g.yfix, N, T, ycmin, ycmax, ycsum, ycount, accumulate, status);
    return launch_status();
}
