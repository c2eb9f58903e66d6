// Weight-only forward  y[t,n] = sum_k x_hat[t,k] w~[n,k] + b[n]  for the ultra-low-bit setting of
// Sec. 4.2 (INT4 / INT3 weights per group along K, FP16 activations): the weight codes are
// de-quantised (Eq. 1: w~ = Step (u - Z)) into binary16 and multiplied on the matrix cores
// (v_mfma_f32_32x32x16_f16, fp32 accumulation).
//
// Two kernels.  dequant_weight_h_kernel writes the binary16 weight [N x K] once per call into
// the caller's workspace: at calibration sizes (hundreds of thousands of tokens) that pass is
// noise, while de-quantising inside the GEMM costs every row tile of tokens the same VALU work
// again (measured: a third of the GEMM's time).  A lane widens two codes at a time into
// binary16 with the 1024 + u trick (the bit pattern 0x6400 | u is the binary16 number
// 1024 + u), subtracts 1024 + Z and multiplies by Step with packed binary16 arithmetic.  Step
// is rounded to binary16 first; for |u - Z| <= 2048 the packed product is the correctly
// rounded binary16 value of (u - Z) Step_h, the value the host-side definition fixes; zero
// points outside [-1024, 1024] take a binary32 path with the same result.
// gemm_f16_kernel: one workgroup of 8 wavefronts (two per SIMD) owns a 256 (t) x 256 (n) output
// tile, each wavefront 128 x 64 of it as 4 x 2 MFMA tiles.  A stage is 64 values of K = 128 bytes
// per row (whole cache lines of both row-major operands), brought in by LDS-DMA loads the
// compiler does not track.  The activation half of a stage goes through a ring of three
// 32 KiB slots (two stages ahead: it misses the L2 twice as often as the weight half and its
// round trip does not fit in one stage), the weight half through two slots; with the
// wavefront's loads retiring in issue order, "at most the 4 newest outstanding" at the end of a
// stage means everything the next stage reads has landed.  The MFMA is issued with the weight
// fragment first so that a lane ends with four consecutive n of one token.  A second form has tiles of
// 128 x 256 (wavefronts of 64 x 64, three slots of both operands) for calls with few tiles.
#include "dequant.hpp"
#include "gemm_wonly_small.hpp"
#include "tile_walk.hpp"
#include <type_traits>

namespace aweq {
namespace wonly {

typedef _Float16 v8h __attribute__((ext_vector_type(8)));
typedef float v16f __attribute__((ext_vector_type(16)));
typedef float v4f __attribute__((ext_vector_type(4)));

constexpr int kThreads = 512;
constexpr int BN = 256;
constexpr int BKH = 64;              // values of K per stage
constexpr int kRow = BKH * 2;        // bytes per tile row per stage
// Tile of 64 MI tokens (MI = 4: 256, MI = 2: 128) x 256 channels in 160 KiB of LDS.  MI = 4: three activation slots, then two
// weight slots.  MI = 2: three slots of both operands (48 KiB), so that the weights run two stages ahead as well.
template <int MI>
struct Tile {
    static constexpr int kRows = 64 * MI;
    static constexpr int kA = kRows * kRow, kB = BN * kRow;         // bytes of a stage's activations, weights
    static constexpr int kStrideA = MI == 4 ? kA : kA + kB;         // slot pitches, and where weight slot 0 starts
    static constexpr int kStrideB = MI == 4 ? kB : kA + kB;
    static constexpr int kFirstB = MI == 4 ? 3 * kA : kA;
    static constexpr int kSlotsB = MI == 4 ? 2 : 3;
    static constexpr int kNewest = MI == 4 ? 4 : 6;                 // loads per wavefront of what is requested last per stage
    static constexpr int kLds = 160 * 1024;
};

// Costs, us at K = 8192: a round of 256-token tiles; one of 128-token tiles against that; the de-quantising pass per channel
constexpr double kTiledRoundCost = 160.0, kHalfTileCost = 0.57, kDequantCost = 0.00445;

struct Args : TileWalk {
    const _Float16* X;     // x_hat [T x K], row-major
    int64_t ldx;
    const _Float16* W;     // de-quantised weight [N x K], row-major (the workspace)
    const float* bias;
    void* out;
    int64_t ldo;
    int64_t T, N, K;
};

// chunk swizzle for 128-byte tile rows: rows sharing LDS banks get distinct chunk positions
// both for 8 and for 16 consecutive rows read at one chunk index
__device__ __forceinline__ int g8(int r) { return (((r >> 1) & 3) << 1) | (((r >> 3) ^ r) & 1); }

// LDS-DMA load the compiler does not track: lane i's 16 bytes land at lds_addr + 16 i
__device__ __forceinline__ void dma16(const char* sbase, uint32_t voff, uint32_t lds_addr)
{
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" ::"s"(lds_addr), "v"(voff), "s"(sbase) : "memory");
}

// A lane turns 8 consecutive codes (4 bytes of INT4; INT3: 24 bits of the 12 bytes a quad of lanes shares) into 16 bytes,
// so that a wavefront stores 1 KiB contiguous; a wavefront takes the same 512 columns of kDqRows rows, whose codes and
// (Step, Z) are all requested before the first is used.  Bound by the write of the binary16 weight: 9.3 us at 4096 x 4096,
// 42 MB.  (With 32 codes per lane, stores 64 bytes apart and two 64-bit divisions per lane it took 24 us.)
constexpr int kDqRows = 4;
template <int BITS>
__global__ __launch_bounds__(256) void dequant_weight_h_kernel(
    const uint8_t* __restrict__ codes, int64_t N, int64_t K, uint32_t chunks, uint32_t scale_pitch, uint32_t group_magic,
    const float* __restrict__ step, const int32_t* __restrict__ zero, _Float16* __restrict__ W)
{
    const int lane = threadIdx.x & (kWave - 1);
    const uint32_t id = blockIdx.x * (256 / kWave) + __builtin_amdgcn_readfirstlane((int)(threadIdx.x / kWave));
    const int64_t n0 = (int64_t)(id / chunks) * kDqRows;
    const uint32_t k = (id % chunks) * (8 * kWave) + lane * 8;
    if (n0 >= N || k >= K) return;
    const int64_t pitch = K / 8 * BITS;
    const uint32_t gi = __umulhi((k & ~31u) >> 4, group_magic);
    uint32_t w[kDqRows];
    float sp[kDqRows];
    int z[kDqRows];
#pragma unroll
    for (int r = 0; r < kDqRows; ++r) {
        const int64_t n = min(n0 + r, N - 1);   // (past the edge: the last row again, not stored)
        const uint8_t* const row = codes + n * pitch;
        if constexpr (BITS == 4) w[r] = *reinterpret_cast<const uint32_t*>(row + k / 2);
        else {
            const uint32_t* const p = reinterpret_cast<const uint32_t*>(row + (k >> 5) * 12);
            const int d = lane & 3;
            w[r] = __builtin_amdgcn_alignbit(p[min(d, 2)], p[max(d - 1, 0)], (32 - 8 * d) & 31);
        }
        sp[r] = step[n * scale_pitch + gi];
        z[r] = zero[n * scale_pitch + gi];
    }
#pragma unroll
    for (int r = 0; r < kDqRows; ++r) {
        if (n0 + r >= N) break;
        Scale<BITS> s;
        s.set(sp[r], z[r]);
        uint32_t o[4];
        if (s.packed) dequant_word<BITS>(w[r], s, o);
        else dequant_word_any<BITS>(w[r], s, o);
        *reinterpret_cast<v4i*>(W + (n0 + r) * K + k) = natural_order(o);
    }
}

#define SB() __builtin_amdgcn_sched_barrier(0)
#define MF(A_, B_, i, j) acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(v8h, B_[j]), __builtin_bit_cast(v8h, A_[i]), acc[i][j], 0, 0, 0)
template <int N>
__device__ __forceinline__ void wait_vm()
{
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
}

// Persistent: the grid is one workgroup per compute unit (a multiple of 8), workgroup b takes the ids
// b, b + grid, b + 2 grid, ...; the first stages of its next tile are requested before the epilogue of
// the current one starts, so the loads fly while the results are stored.
template <int MI, bool OUT_F16>
__global__ __launch_bounds__(kThreads) void gemm_f16_kernel(Args g)
{
    using TL = Tile<MI>;
    extern __shared__ __attribute__((aligned(1024))) char lds[];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int wm = wave >> 2, wn = wave & 3;
    const int stride = gridDim.x;

    int vb = blockIdx.x, tile_m = 0, tile_n = 0;
    while (vb < g.n_ids && !tile_of(g, vb, tile_m, tile_n)) vb += stride;
    if (vb >= g.n_ids) return;

    const int ns = (int)(g.K / BKH);
    const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char*)lds;
    const uint32_t wave_offA = __builtin_amdgcn_readfirstlane(wave) * (1024 * MI), wave_offB = TL::kFirstB + __builtin_amdgcn_readfirstlane(wave) * 4096;

    // fragment of K-step qq (16 values = 32 bytes per row): lane reads row lane % 32 of a 32-row
    // sub-tile, chunk 2 qq + lane / 32
    const int fr_row = lane & 31, fr_half = lane >> 5;
    const int fsw = g8(fr_row);
    int offA[4], offB[4];
#pragma unroll
    for (int qq = 0; qq < 4; ++qq) {
        offA[qq] = (wm * (32 * MI) + fr_row) * kRow + ((qq * 2 + fr_half) ^ fsw) * 16;
        offB[qq] = TL::kFirstB + (wn * 64 + fr_row) * kRow + ((qq * 2 + fr_half) ^ fsw) * 16;
    }

    // global -> LDS: wave w brings tile rows 32 w .. 32 w + 31 of the weight and 8 MI w .. of the activations, 8 rows x
    // 128 B per instruction; lane i sits at row i / 8, chunk slot i % 8 and fetches chunk slot ^ g8(row)
    const char* baseA;   // the tile's first rows (wave-uniform: scalar registers)
    const char* baseB;
    uint32_t oa[MI], ob[4];  // byte offsets from the tile's first row: < 256 * 2 ldx
    int64_t m0, n0;

#define RDA(dst, qq, i) dst[i] = *reinterpret_cast<const v4i*>(sa + offA[qq] + (i) * 32 * kRow)
#define RDB(dst, qq, j) dst[j] = *reinterpret_cast<const v4i*>(sb + offB[qq] + (j) * 32 * kRow)
#define DMA_A(q, s_) dma16(baseA + (int64_t)(s_) * kRow, oa[q], lds0 + ((s_) % 3) * TL::kStrideA + wave_offA + (q) * 1024)
#define DMA_B(q, s_) dma16(baseB + (int64_t)(s_) * kRow, ob[q], lds0 + ((s_) % TL::kSlotsB) * TL::kStrideB + wave_offB + (q) * 1024)

    // addresses of tile (tm, tn); stage 0 of both operands and what of stage 1 runs two stages ahead on their way
    auto start_tile = [&](int tm, int tn) {
        m0 = (int64_t)__builtin_amdgcn_readfirstlane(tm) * TL::kRows;
        n0 = (int64_t)__builtin_amdgcn_readfirstlane(tn) * BN;
        baseA = reinterpret_cast<const char*>(g.X + m0 * g.ldx);
        baseB = reinterpret_cast<const char*>(g.W + n0 * g.K);
        // rows past the edge re-read the last valid row; their results are never stored
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            if (q < MI) {
                const int row = wave * (8 * MI) + q * 8 + (lane >> 3);
                oa[q] = (uint32_t)((min(m0 + row, g.T - 1) - m0) * g.ldx * 2 + ((lane & 7) ^ g8(row)) * 16);
            }
            const int row = wave * 32 + q * 8 + (lane >> 3);
            ob[q] = (uint32_t)((min(n0 + row, g.N - 1) - n0) * g.K * 2 + ((lane & 7) ^ g8(row)) * 16);
        }
#pragma unroll
        for (int q = 0; q < MI; ++q) DMA_A(q, 0);
#pragma unroll
        for (int q = 0; q < 4; ++q) DMA_B(q, 0);
        if (ns > 1) {
#pragma unroll
            for (int q = 0; q < MI; ++q) DMA_A(q, 1);
            if constexpr (MI == 2) {
#pragma unroll
                for (int q = 0; q < 4; ++q) DMA_B(q, 1);
            }
        }
    };

    start_tile(tile_m, tile_n);
    if (ns > 1) wait_vm<TL::kNewest>(); else wait_vm<0>();

    // Vector memory operations of a wave complete in the order issued.  A tile that lies inside the
    // output issues 8 MI stores per wave after requesting the next tile's first stages, so "at most
    // that many + kNewest operations pending" means stage 0 has landed while the stores (and the loads
    // of stage 1) may still be on their way.
    constexpr int kStores = 8 * MI;

    for (;;) {
        const int64_t cm0 = m0, cn0 = n0;   // the tile being multiplied
        v16f acc[MI][2];
#pragma unroll
        for (int i = 0; i < MI; ++i)
#pragma unroll
            for (int j = 0; j < 2; ++j)
#pragma unroll
                for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.0f;
        v4i a0[MI], b0[2], a1[MI], b1[2];

        __builtin_amdgcn_s_barrier();   // stage 0 has landed for every wave
        {
            const char* sa = lds;
            const char* sb = lds;
#pragma unroll
            for (int i = 0; i < MI; ++i) RDA(a0, 0, i);
            RDB(b0, 0, 0); RDB(b0, 0, 1);
        }

        // one stage (64 values of K) = four K-steps of 2 MI MFMAs per wave.  F0 / F1 are the two fragment
        // register sets; each K-step multiplies one and fetches the other.  NEXT: there is a stage
        // s + 1 (MI = 4: its weights are requested here); NEXT2: there is a stage s + 2 (its activations, and
        // for MI = 2 its weights, are).  The slots of stage s - 1, which these loads go to, are free: every wave
        // passed that stage's barrier.
        auto stage = [&](int s, auto next_c, auto next2_c) {
            constexpr bool NEXT = decltype(next_c)::value;
            constexpr bool NEXT2 = decltype(next2_c)::value;
            const char* sa = lds + (s % 3) * TL::kStrideA;
            const char* sb = lds + (s % TL::kSlotsB) * TL::kStrideB;
            // K-step 0: multiply F0, fetch F1
            SB();
            if constexpr (MI == 4) {
                RDA(a1, 1, 0); RDB(b1, 1, 0); RDB(b1, 1, 1); MF(a0, b0, 0, 0);
                SB();
                if constexpr (NEXT) DMA_B(0, s + 1);
                RDA(a1, 1, 1); RDA(a1, 1, 2); MF(a0, b0, 0, 1);
                SB();
                if constexpr (NEXT) DMA_B(1, s + 1);
                RDA(a1, 1, 3); MF(a0, b0, 1, 0);
                SB();
                if constexpr (NEXT) DMA_B(2, s + 1);
                MF(a0, b0, 1, 1);
                SB();
                if constexpr (NEXT) DMA_B(3, s + 1);
                MF(a0, b0, 2, 0); MF(a0, b0, 2, 1); MF(a0, b0, 3, 0); MF(a0, b0, 3, 1);
                SB();
                // K-step 1: multiply F1, fetch F0
                RDA(a0, 2, 0); RDB(b0, 2, 0); RDB(b0, 2, 1); MF(a1, b1, 0, 0);
                SB();
                if constexpr (NEXT2) DMA_A(0, s + 2);
                RDA(a0, 2, 1); RDA(a0, 2, 2); MF(a1, b1, 0, 1);
                SB();
                if constexpr (NEXT2) DMA_A(1, s + 2);
                RDA(a0, 2, 3); MF(a1, b1, 1, 0);
                SB();
                if constexpr (NEXT2) DMA_A(2, s + 2);
                MF(a1, b1, 1, 1);
                SB();
                if constexpr (NEXT2) DMA_A(3, s + 2);
                MF(a1, b1, 2, 0); MF(a1, b1, 2, 1); MF(a1, b1, 3, 0); MF(a1, b1, 3, 1);
                SB();
                // K-step 2: multiply F0, fetch F1
                RDA(a1, 3, 0); RDB(b1, 3, 0); RDB(b1, 3, 1); MF(a0, b0, 0, 0);
                SB();
                RDA(a1, 3, 1); RDA(a1, 3, 2); MF(a0, b0, 0, 1);
                SB();
                RDA(a1, 3, 3); MF(a0, b0, 1, 0);
                SB();
                MF(a0, b0, 1, 1); MF(a0, b0, 2, 0); MF(a0, b0, 2, 1); MF(a0, b0, 3, 0); MF(a0, b0, 3, 1);
                SB();
            } else {
                RDA(a1, 1, 0); RDB(b1, 1, 0); MF(a0, b0, 0, 0);
                SB();
                if constexpr (NEXT2) DMA_A(0, s + 2);
                RDB(b1, 1, 1); RDA(a1, 1, 1); MF(a0, b0, 0, 1);
                SB();
                if constexpr (NEXT2) DMA_A(1, s + 2);
                MF(a0, b0, 1, 0);
                SB();
                if constexpr (NEXT2) DMA_B(0, s + 2);
                MF(a0, b0, 1, 1);
                SB();
                // K-step 1: multiply F1, fetch F0
                RDA(a0, 2, 0); RDB(b0, 2, 0); MF(a1, b1, 0, 0);
                SB();
                if constexpr (NEXT2) DMA_B(1, s + 2);
                RDB(b0, 2, 1); RDA(a0, 2, 1); MF(a1, b1, 0, 1);
                SB();
                if constexpr (NEXT2) DMA_B(2, s + 2);
                MF(a1, b1, 1, 0);
                SB();
                if constexpr (NEXT2) DMA_B(3, s + 2);
                MF(a1, b1, 1, 1);
                SB();
                // K-step 2: multiply F0, fetch F1
                RDA(a1, 3, 0); RDB(b1, 3, 0); MF(a0, b0, 0, 0);
                SB();
                RDB(b1, 3, 1); RDA(a1, 3, 1); MF(a0, b0, 0, 1);
                SB();
                MF(a0, b0, 1, 0); MF(a0, b0, 1, 1);
                SB();
            }
            if constexpr (NEXT) {
                // stage s + 1 has landed for this wave (only the kNewest loads issued last, of stage
                // s + 2, may still be out), its reads of stage s are done; after the barrier that holds
                // for every wave
                if constexpr (NEXT2) wait_vm<TL::kNewest>(); else wait_vm<0>();
                asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
                __builtin_amdgcn_s_barrier();
                SB();
                sa = lds + ((s + 1) % 3) * TL::kStrideA;
                sb = lds + ((s + 1) % TL::kSlotsB) * TL::kStrideB;
                // K-step 3: multiply F1, fetch F0 = K-step 0 of the next stage
                if constexpr (MI == 4) {
                    RDA(a0, 0, 0); RDB(b0, 0, 0); RDB(b0, 0, 1); MF(a1, b1, 0, 0);
                    SB();
                    RDA(a0, 0, 1); RDA(a0, 0, 2); MF(a1, b1, 0, 1);
                    SB();
                    RDA(a0, 0, 3); MF(a1, b1, 1, 0);
                    SB();
                    MF(a1, b1, 1, 1); MF(a1, b1, 2, 0); MF(a1, b1, 2, 1); MF(a1, b1, 3, 0); MF(a1, b1, 3, 1);
                } else {
                    RDA(a0, 0, 0); RDB(b0, 0, 0); MF(a1, b1, 0, 0);
                    SB();
                    RDB(b0, 0, 1); RDA(a0, 0, 1); MF(a1, b1, 0, 1);
                    SB();
                    MF(a1, b1, 1, 0); MF(a1, b1, 1, 1);
                }
                SB();
            } else {
#pragma unroll
                for (int i = 0; i < MI; ++i) { MF(a1, b1, i, 0); MF(a1, b1, i, 1); }
            }
        };
        int s = 0;
        for (; s + 2 < ns; ++s) stage(s, std::true_type{}, std::true_type{});
        if (s + 1 < ns) { stage(s, std::true_type{}, std::false_type{}); ++s; }
        stage(s, std::false_type{}, std::false_type{});

        // ---- epilogue.  With the weight fragment as first MFMA operand, register v of lane l in
        // sub-tile (i, j) is token t = m0 + 32 MI wm + 32 i + l % 32 and output channel
        // n = n0 + 64 wn + 32 j + 8 (v / 4) + 4 (l / 32) + v % 4.  Each wave turns its 32 (t) x 64 (n)
        // slab of sub-tile row i around in a private 8 KiB LDS region (256-byte rows, XOR-swizzled
        // 16-byte chunks) so that 16 lanes cover one output row of the slab per store.  The slabs live
        // in the third activation slot and the second weight slot (MI = 2: in the third slot and behind it): the
        // next tile's first stages are already on their way into the others.
        const int wr_t = lane & 31, wr_sw = wr_t & 15, wr_half = lane >> 5;
        const int rd_r = lane >> 4, rd_c = lane & 15;
        const int64_t n = cn0 + wn * 64 + rd_c * 4;      // this lane's four channels
        const bool n_ok = n < g.N;                       // N % 4 == 0: all four or none
        const int64_t t_lane = cm0 + wm * (32 * MI) + rd_r;    // + 32 i + 4 p
        // what the epilogue reads from memory is requested before the next tile's stages, so that
        // waiting for it does not wait for them (pinned: the compiler's wait then sits here)
        v4f bs = {0.f, 0.f, 0.f, 0.f};
        if (g.bias && n_ok) bs = *reinterpret_cast<const v4f*>(g.bias + n);
#pragma unroll
        for (int c = 0; c < 4; ++c) asm volatile("" : "+v"(bs[c]));

        // next tile of this workgroup
        int nvb = vb + stride, ntm = 0, ntn = 0;
        while (nvb < g.n_ids && !tile_of(g, nvb, ntm, ntn)) nvb += stride;
        const bool more = nvb < g.n_ids;
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        __builtin_amdgcn_s_barrier();   // every wave is done reading the stage buffers
        if (more) start_tile(ntm, ntn);

        char* slab = lds + (MI == 2 ? 2 * TL::kStrideA + wave * 8192 : wave < 4 ? 2 * TL::kA + wave * 8192 : TL::kFirstB + TL::kB + (wave - 4) * 8192);
#pragma unroll
        for (int i = 0; i < MI; ++i) {
#pragma unroll
            for (int j = 0; j < 2; ++j)
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    v4f o = {acc[i][j][4 * q], acc[i][j][4 * q + 1], acc[i][j][4 * q + 2], acc[i][j][4 * q + 3]};
                    *reinterpret_cast<v4f*>(slab + wr_t * 256 + (((8 * j + 2 * q + wr_half) ^ wr_sw) * 16)) = o;
                }
#pragma unroll
            for (int p = 0; p < 8; ++p) {
                const int r = 4 * p + rd_r;
                v4f o = *reinterpret_cast<const v4f*>(slab + r * 256 + ((rd_c ^ (r & 15)) * 16));
                const int64_t t = t_lane + i * 32 + 4 * p;
                if (t < g.T && n_ok) {
                    o += bs;
                    if constexpr (OUT_F16) {
                        typedef _Float16 h4 __attribute__((ext_vector_type(4)));
                        h4 oh = {(_Float16)o[0], (_Float16)o[1], (_Float16)o[2], (_Float16)o[3]};
                        __builtin_nontemporal_store(oh, reinterpret_cast<h4*>(reinterpret_cast<_Float16*>(g.out) + t * g.ldo + n));
                    } else {
                        __builtin_nontemporal_store(o, reinterpret_cast<v4f*>(reinterpret_cast<float*>(g.out) + t * g.ldo + n));
                    }
                }
            }
        }
        if (!more) break;
        vb = nvb;
        // stage 0 of the next tile has landed (interior tile: its stores may still drain)
        if (ns > 1 && cm0 + TL::kRows <= g.T && cn0 + BN <= g.N) wait_vm<kStores + TL::kNewest>();
        else wait_vm<0>();
    }
#undef RDA
#undef RDB
#undef DMA_A
#undef DMA_B
}
#undef SB
#undef MF

}  // namespace wonly
}  // namespace aweq

using namespace aweq;

extern "C" int aweq_wonly_gemm(const void* X_hat, int64_t T, int64_t K, int64_t ldx,
                               const void* codes, int bits, int group,
                               const float* step_w, const int32_t* zero_w, int64_t N,
                               const float* bias, void* out, aweq_dtype out_dt, int64_t ldo,
                               void* ws, size_t ws_bytes, uint32_t* status, void* stream)
{
    (void)status;
    if (!X_hat || !codes || !step_w || !zero_w || !out) return AWEQ_ERR_NULL;
    if (bits != 4 && bits != 3) return AWEQ_ERR_BITS;
    if (out_dt != AWEQ_F16 && out_dt != AWEQ_F32) return AWEQ_ERR_DTYPE;
    if (T <= 0 || N <= 0 || K <= 0 || (K % wonly::BKH) != 0 || ldx < K || ldo < N) return AWEQ_ERR_SHAPE;
    if (K > (1 << 20)) return AWEQ_ERR_SHAPE;  // 32-bit byte offsets inside a tile of rows
    if (group < -1 || (group > 0 && ((group % 32) != 0 || (K % group) != 0))) return AWEQ_ERR_GROUP;
    if ((N % 4) != 0 || (ldo % 4) != 0) return AWEQ_ERR_SHAPE;
    if (!aligned16(X_hat) || (ldx % 8) != 0 || !aligned16(codes) || !aligned16(out) || (bias && !aligned16(bias)))
        return AWEQ_ERR_ALIGN;
    if (!ws || ws_bytes < (size_t)N * (size_t)K * 2) return AWEQ_ERR_WORKSPACE;
    if (!aligned16(ws)) return AWEQ_ERR_ALIGN;
    hipStream_t st = as_stream(stream);

    const uint32_t scale_pitch = group < 0 ? 0u : group == 0 ? 1u : (uint32_t)(K / group);
    const uint32_t group_magic = group <= 0 ? 0u : (uint32_t)cdiv(1ll << 31, group / 32);
    const bool f16 = out_dt == AWEQ_F16;
    // An output over an input: the codes and their (Step, Z) are read by the de-quantising pass, before the GEMM stores anything, and
    // with up to 256 channels a row of X_hat by the workgroup that stores that row (one tile of 256 tokens: everything).  Straight from
    // the codes a workgroup would store over what another still reads.
    const int64_t scales = group < 0 ? 4 : group == 0 ? N * 4 : N * (K / group) * 4;
    const Span o = matrix_span(out, T, N, ldo, dtype_size(out_dt));
    const bool apart = !overlap({o}, {{codes, N * (K / 8 * bits)}, {step_w, scales}, {zero_w, scales}}) &&
                       (N > 256 || !overlap({o}, {matrix_span(X_hat, T, K, ldx, 2), {bias, N * 4}}));
    // tiles of 256 tokens, or of 128 where their rounds of workgroups take less: a round lasts as long however few of the 256
    // compute units have a tile (GEMM alone, us, 256 -> 128 tokens a tile: 1531 tokens 4096 x 4096 78 -> 51, 4096 x 11008 226 -> 126,
    // 768 tokens 8192 x 8192 164 -> 90)
    wonly::Args g, h;
    int64_t blocks = 0;
    int rc = plan_walk(g, T, N, K, 256, blocks);
    if (rc != AWEQ_OK) return rc;
    // Byte offsets inside a tile of rows are 32-bit: whether they reach the last of `rows` tokens (512: a stage's bytes of a row)
    auto reach = [&](int64_t rows) { return (T < rows ? T : rows) - 1 <= (((1ll << 32) - 512) / 2) / ldx; };
    const bool half = plan_walk(h, T, N, K, 128, blocks) == AWEQ_OK && ((apart && wonly::kHalfTileCost * (double)rounds_of(h) < (double)rounds_of(g)) || !reach(256));
    const double tiled_cost = (half ? wonly::kHalfTileCost * (double)rounds_of(h) : (double)rounds_of(g)) * wonly::kTiledRoundCost + wonly::kDequantCost * (double)N;
    if (half) g = h;

    // Straight from the codes where one of the two kernels that do so is modelled to take less (both sides measured in
    // gemm_wonly_small.hip and gemm_wonly_mid.hip).
    wonly::SmallArgs a;
    a.X = reinterpret_cast<const _Float16*>(X_hat); a.codes = reinterpret_cast<const uint8_t*>(codes);
    a.step = step_w; a.zero = zero_w; a.bias = bias; a.out = out; a.ldx = ldx; a.ldo = ldo; a.T = T; a.N = N; a.K = K;
    a.scale_pitch = scale_pitch;
    a.group_magic = group_magic;
    wonly::SmallPlan small = wonly::plan_small(T, N);
    // The few-token kernel's time falls more slowly with K than the others' (its wavefronts take 256 values each, and however few have some,
    // eight partial sums are added; us, groups of 64, it / the tiled form: 100 tokens 32000 x 4096 126 / 137, x 1024 56 / 35, x 256
    // 43 / 21; 512 tokens 4096 x 768 23.7 / 17.7, x 256 22.8 / 11.7)
    if (K < 8192) small.cost *= (double)(K + 1024) / (double)(K + 384) * (8192.0 + 384.0) / (8192.0 + 1024.0);
    const wonly::MidPlan mid = wonly::plan_mid(T, N);
    const bool tiled_ok = reach(half ? 128 : 256), mid_ok = apart && (group <= 0 || group % 128 == 0) && reach(128);
    // the de-quantising pass is a launch more, about 0.6 us of such small calls (312 tokens 2532 x 64, groups of 64, 8.3 / 9.6)
    const double launch_cost = 0.6 * 8192.0 / (double)K;
    if (!tiled_ok || (apart && small.cost <= tiled_cost + launch_cost && (!mid_ok || small.cost <= mid.cost))) {
        // Its token tiles ride on the grid's y dimension, 65535 of 32 tokens to a launch, and its 32-bit offsets count elements: of
        // pitches beyond their reach (2^27 for a tile of 32 tokens) a launch takes the tokens that they reach.
        const int64_t last = ((1ll << 32) - 1 - K) / ldx, step = last >= 31 ? 65535 * 32 : last + 1;
        for (int64_t t = 0; t < T; t += step) {
            a.T = T - t < step ? T - t : step;
            a.X = reinterpret_cast<const _Float16*>(X_hat) + t * ldx;
            a.out = reinterpret_cast<char*>(out) + t * ldo * (int64_t)dtype_size(out_dt);
            rc = wonly::launch_small(a, bits, group, small, f16, st);
            if (rc != AWEQ_OK) return rc;
        }
        return AWEQ_OK;
    }
    if (mid_ok && mid.cost <= tiled_cost) return wonly::launch_mid(a, bits, mid, f16, st);

    // the binary16 weight, once
    _Float16* W = reinterpret_cast<_Float16*>(ws);
    const uint32_t chunks = (uint32_t)cdiv(K, 8 * kWave);
    const int64_t dq_blocks = cdiv(cdiv(N, wonly::kDqRows) * chunks, 256 / kWave);
    if (dq_blocks > 0x3fffffffll) return AWEQ_ERR_SHAPE;
    const uint8_t* cb = reinterpret_cast<const uint8_t*>(codes);
    if (bits == 4) wonly::dequant_weight_h_kernel<4><<<(unsigned)dq_blocks, 256, 0, st>>>(cb, N, K, chunks, scale_pitch, group_magic, step_w, zero_w, W);
    else wonly::dequant_weight_h_kernel<3><<<(unsigned)dq_blocks, 256, 0, st>>>(cb, N, K, chunks, scale_pitch, group_magic, step_w, zero_w, W);

    g.X = reinterpret_cast<const _Float16*>(X_hat); g.ldx = ldx;
    g.W = W; g.bias = bias;
    g.out = out; g.ldo = ldo; g.T = T; g.N = N; g.K = K;
    const void* fn = half ? (f16 ? reinterpret_cast<const void*>(wonly::gemm_f16_kernel<2, true>) : reinterpret_cast<const void*>(wonly::gemm_f16_kernel<2, false>))
                          : (f16 ? reinterpret_cast<const void*>(wonly::gemm_f16_kernel<4, true>) : reinterpret_cast<const void*>(wonly::gemm_f16_kernel<4, false>));
    return launch_persistent(fn, wonly::kThreads, wonly::Tile<4>::kLds, &g, g.n_ids, st);
}
