// Stage 3: asymmetric round-to-nearest weight quantizer (Sec. 2, Eq. 1-2) with the three
// storage formats (int8, packed 4-bit, packed 3-bit).
//
// HBM-bound: each weight is read once and its code written once.  A thread owns "units" of
// 8 consecutive k (16 bytes of binary16, 32 bytes of binary32).  Per-row slices keep the
// whole row in registers between the min/max reduction and the quantization; per-group
// slices are 2^m lanes wide and reduce with DPP butterflies only.
#include "weight_unit.hpp"

namespace aweq {

constexpr int kQwBlock = 256;
constexpr int kQwMaxUnits = 12;  // units per thread held in registers: K <= 256 * 8 * 12 = 24576

// ---- one (Step, Z) per row, or one for the tensor (PER_TENSOR: read from step[0]/zero[0]).
// 8-bit codes are the GEMM's weight operand and go out in its K-panel layout.
// FOLD: the row read is the un-equalised W; it is multiplied by s[k] (one fp32 multiply, rounded to
// the weight's type: Eq. 3), written to W_hat and quantised from registers, so W is read once.
// TPR threads hold a whole row in UPT units per thread, all requested before the first is used.  Bound by memory (fold and
// quantise, binary16, us, with the division and the units one after the other -> now: 4096 x 4096 26.6 -> 23.0, 4096 x 11008
// 58.1 -> 47.5, 225 MB; several rows per block, or neighbouring rows on one XCD, gain nothing).
template <bool F16, int BITS, bool PER_TENSOR, bool FOLD, int TPR, int UPT>
__global__ __launch_bounds__(kQwBlock) void quant_weight_row(
    const void* __restrict__ W, int64_t N, int64_t K, int64_t ldw, uint8_t* __restrict__ codes,
    float* __restrict__ step, int32_t* __restrict__ zero, int32_t* __restrict__ rowsum_w, uint32_t* status,
    const float* __restrict__ s, void* __restrict__ W_hat, int64_t ldwh)
{
    constexpr int kRows = kQwBlock / TPR;        // rows per block: one, or one per wavefront
    __shared__ float slot_f[kQwBlock / kWave];
    __shared__ int slot_i[kQwBlock / kWave];
    const int tid = threadIdx.x % TPR;
    const int64_t n = (int64_t)blockIdx.x * kRows + threadIdx.x / TPR;
    if (kRows > 1 && n >= N) return;             // (no barriers when rows sit in wavefronts)
    const int64_t units = K / 8;
    const char* const row = reinterpret_cast<const char*>(W) + (size_t)n * ldw * (F16 ? 2 : 4);
    char* const row_hat = reinterpret_cast<char*>(W_hat) + (size_t)n * ldwh * (F16 ? 2 : 4);
    uint8_t* const row_codes = BITS == 8 ? codes + (size_t)n * kPanel : codes + (size_t)n * (K * BITS / 8);
    auto reduce = [](auto v, auto op, auto* slot) {
        if constexpr (TPR == kWave) return wave_allreduce(v, op);
        else return block_allreduce<kQwBlock / kWave>(v, op, slot);
    };
    uint32_t st = 0;

    Unit<F16> reg[UPT];
#pragma unroll
    for (int j = 0; j < UPT; ++j) {
        const int64_t u = tid + (int64_t)j * TPR;
        if (u < units) reg[j].load(row, u);
    }
    Extremes<F16> ex;
#pragma unroll
    for (int j = 0; j < UPT; ++j) {
        const int64_t u = tid + (int64_t)j * TPR;
        if (u < units) {
            if constexpr (FOLD) {
                float x[8];
                reg[j].get(x);
                const Float4 s0 = *reinterpret_cast<const Float4*>(s + u * 8), s1 = *reinterpret_cast<const Float4*>(s + u * 8 + 4);
#pragma unroll
                for (int i = 0; i < 4; ++i) { x[i] = rounded_f32(x[i] * s0.f[i]); x[4 + i] = rounded_f32(x[4 + i] * s1.f[i]); }
                reg[j].set(x);
                reg[j].store(row_hat, u);
            }
            ex.add(reg[j]);
        }
    }
    float sp;
    int z;
    if constexpr (PER_TENSOR) {
        sp = step[0];
        z = zero[0];
    } else {
        const float lo = reduce(ex.min(), OpMin(), slot_f);
        const float hi = reduce(ex.max(), OpMax(), slot_f);
        qparams(lo, hi, BITS, sp, z, st);
        if (tid == 0) { step[n] = sp; zero[n] = z; }
    }
    const ActParams p = quot_params(sp, z);
    const bool screened = __all(may_screen(ex, p));
    int rs = 0;
#pragma unroll
    for (int j = 0; j < UPT; ++j) {
        const int64_t u = tid + (int64_t)j * TPR;
        if (u < units) {
            float x[8];
            reg[j].get(x);
            // unit u of row n in the panel layout: panel u / 8, bytes 8 (u % 8) ..
            rs += quant_store_unit<BITS>(x, p, screened, row_codes, u, st, BITS == 8 ? (u >> 3) * N * kPanel + (u & 7) * 8 : -1);
        }
    }
    if constexpr (BITS == 8) {
        // columns past K in the last panel are zero
        const int64_t u = units + tid;
        if (u < panel_count(K) * 8) *reinterpret_cast<uint2*>(row_codes + (u >> 3) * N * kPanel + (u & 7) * 8) = make_uint2(0u, 0u);
    }
    if (BITS == 8 && rowsum_w) {
        rs = reduce(rs, OpAdd(), slot_i);
        if (tid == 0) rowsum_w[n] = rs;
    }
    raise_status(status, st);
}

// ---- one (Step, Z) per group of 8 * 2^LEVELS consecutive k inside a row.  Large binary16 calls are bound by the vector unit: the
// slice's three divisions and its reductions cost as much as quantising a unit, so a lane takes UNITS = 2 units of a group (from 64
// values on) and a thread the same units of ROWS = 2 rows.  Small calls are one chain of dependent steps, which must not be longer than
// one unit needs, and binary32 is bound by its loads, which want more and simpler threads (rule and figures at the launch).
template <bool F16, int BITS, int LEVELS, int ROWS, int UNITS>
__global__ __launch_bounds__(kQwBlock) void quant_weight_group(
    const void* __restrict__ W, int64_t N, int64_t K, int64_t ldw, uint8_t* __restrict__ codes,
    float* __restrict__ step, int32_t* __restrict__ zero, uint32_t* status)
{
    constexpr int kUnits = LEVELS >= 3 ? UNITS : 1, kLanes = LEVELS - (kUnits - 1);   // units per lane; 2^kLanes lanes per group
    const int64_t n0 = (int64_t)blockIdx.y * ROWS;
    const int64_t units = K / 8;
    const int64_t id = (int64_t)blockIdx.x * kQwBlock + threadIdx.x, g = id >> kLanes;
    const int64_t u0 = (g << LEVELS) + (id & ((1 << kLanes) - 1));
    // K % group == 0 and groups are lane-aligned, so a group is entirely in or out of range
    if (u0 >= units) return;
    uint32_t st = 0;
    Unit<F16> reg[ROWS][kUnits];
#pragma unroll
    for (int i = 0; i < ROWS; ++i)   // (past the edge: the last row again, not stored)
#pragma unroll
        for (int j = 0; j < kUnits; ++j)
            reg[i][j].load(reinterpret_cast<const char*>(W) + (size_t)min(n0 + i, N - 1) * ldw * (F16 ? 2 : 4), u0 + (j << kLanes));
#pragma unroll
    for (int i = 0; i < ROWS; ++i) {
        const int64_t n = n0 + i;
        if (n >= N) break;
        Extremes<F16> ex;
#pragma unroll
        for (int j = 0; j < kUnits; ++j) ex.add(reg[i][j]);
        const float lo = group_allreduce<kLanes>(ex.min(), OpMin());
        const float hi = group_allreduce<kLanes>(ex.max(), OpMax());
        float sp;
        int z;
        qparams(lo, hi, BITS, sp, z, st);
        const ActParams p = quot_params(sp, z);
        const bool screened = __all(may_screen(ex, p));
#pragma unroll
        for (int j = 0; j < kUnits; ++j) {
            float x[8];
            reg[i][j].get(x);
            quant_store_unit<BITS>(x, p, screened, codes + (size_t)n * (K * BITS / 8), u0 + (j << kLanes), st);
        }
        if ((id & ((1 << kLanes) - 1)) == 0) {
            const int64_t gi = n * (units >> LEVELS) + g;
            step[gi] = sp;
            zero[gi] = z;
        }
    }
    raise_status(status, st);
}

// ---- tensor-wide extremes for group = -1: order-preserving unsigned keys + atomics
__device__ __forceinline__ uint32_t float_key(float f)
{
    uint32_t b = __float_as_uint(f);
    return (b & 0x80000000u) ? ~b : (b | 0x80000000u);
}
__device__ __forceinline__ float key_float(uint32_t k)
{
    return __uint_as_float((k & 0x80000000u) ? (k & 0x7fffffffu) : ~k);
}

__global__ void tensor_minmax_init(uint32_t* keys)
{
    keys[0] = 0xffffffffu;  // running minimum
    keys[1] = 0u;           // running maximum
}

template <bool F16>
__global__ __launch_bounds__(kQwBlock) void tensor_minmax(const void* __restrict__ W, int64_t N, int64_t K,
                                                          int64_t ldw, uint32_t* keys)
{
    __shared__ float slot[kQwBlock / kWave];
    const int64_t units = K / 8;
    float lo = INFINITY, hi = -INFINITY;
    for (int64_t n = blockIdx.x; n < N; n += gridDim.x) {
        const char* row = reinterpret_cast<const char*>(W) + (size_t)n * ldw * (F16 ? 2 : 4);
        for (int64_t u = threadIdx.x; u < units; u += kQwBlock) {
            Unit<F16> reg;
            reg.load(row, u);
            float x[8];
            reg.get(x);
            minmax8(x, lo, hi);
        }
    }
    lo = block_allreduce<kQwBlock / kWave>(lo, OpMin(), slot);
    hi = block_allreduce<kQwBlock / kWave>(hi, OpMax(), slot);
    if (threadIdx.x == 0) {
        atomicMin(&keys[0], float_key(lo));
        atomicMax(&keys[1], float_key(hi));
    }
}

__global__ void tensor_qparams(const uint32_t* keys, int bits, float* step, int32_t* zero, uint32_t* status)
{
    uint32_t st = 0;
    float sp;
    int z;
    qparams(key_float(keys[0]), key_float(keys[1]), bits, sp, z, st);
    *step = sp;
    *zero = z;
    raise_status(status, st);
}

// Rows of up to 1024 values sit in a wavefront each (512 x 512 binary32: 4.0 -> 3.4 us), up to 4096 in two units per thread
// (4096 x 4096 binary16: 24.7 us with the registers of twelve, 23.0 with two)
template <bool F16, int BITS, bool PER_TENSOR, bool FOLD>
static void launch_row(const void* W, int64_t N, int64_t K, int64_t ldw, uint8_t* codes, float* step, int32_t* zero, int32_t* rowsum_w,
                       uint32_t* status, hipStream_t st, const float* s = nullptr, void* W_hat = nullptr, int64_t ldwh = 0)
{
#define AWEQ_QR(TPR, UPT)                                                                                              \
    quant_weight_row<F16, BITS, PER_TENSOR, FOLD, TPR, UPT><<<(unsigned)cdiv(N, kQwBlock / TPR), kQwBlock, 0, st>>>(   \
        W, N, K, ldw, codes, step, zero, rowsum_w, status, s, W_hat, ldwh)
    if (K <= 1024) AWEQ_QR(64, 2);
    else if (K <= 4096) AWEQ_QR(256, 2);
    else AWEQ_QR(256, kQwMaxUnits);
#undef AWEQ_QR
}

template <bool F16, int BITS, int ROWS, int UNITS>
static void launch_group_as(int levels, const void* W, int64_t N, int64_t K, int64_t ldw, uint8_t* codes,
                            float* step, int32_t* zero, uint32_t* status, hipStream_t st)
{
    dim3 grid((unsigned)cdiv(levels >= 3 ? K / (8 * UNITS) : K / 8, kQwBlock), (unsigned)cdiv(N, ROWS));
#define AWEQ_LG(L) case L: quant_weight_group<F16, BITS, L, ROWS, UNITS><<<grid, kQwBlock, 0, st>>>(W, N, K, ldw, codes, step, zero, status); break;
    switch (levels) { AWEQ_LG(0) AWEQ_LG(1) AWEQ_LG(2) AWEQ_LG(3) AWEQ_LG(4) AWEQ_LG(5) AWEQ_LG(6) }
#undef AWEQ_LG
}

// Rows x units of a thread (us, groups of 128, 4 bits, 1 x 1 / 2 x 1 / 2 x 2): binary16 from 2^22 values on two by two (4096 x 11008 34.7 / 33.0 /
// 24.2, 11008 x 11008 89.8 / 82.6 / 56.4), fewer one by one (512 x 512 3.4 / 3.7 / 4.4, 64 x 4096 3.3 / 3.8 / 4.1).  Binary32 one by one
// (11008 x 5120 46.8 / 48.6 / 55.2, 4096 x 22016 74.2 / 75.9 / 84.5).  Rows of up to 512 values leave most of a block without
// work: from 8192 rows on two rows a thread (11008 x 256 in groups of 8 7.6 / 6.0 / 6.0, 11008 x 512 8.2 / 8.0 / 9.3; but 4096 x 512 4.8 / 5.1 / 5.5).
template <bool F16, int BITS>
static void launch_group(int levels, const void* W, int64_t N, int64_t K, int64_t ldw, uint8_t* codes,
                         float* step, int32_t* zero, uint32_t* status, hipStream_t st)
{
    if (K <= 512 && N >= 8192) launch_group_as<F16, BITS, 2, 1>(levels, W, N, K, ldw, codes, step, zero, status, st);
    else if (F16 && K > 512 && N * K >= (1ll << 22)) launch_group_as<F16, BITS, 2, F16 ? 2 : 1>(levels, W, N, K, ldw, codes, step, zero, status, st);
    else launch_group_as<F16, BITS, 1, 1>(levels, W, N, K, ldw, codes, step, zero, status, st);
}

}  // namespace aweq

using namespace aweq;

extern "C" int aweq_quant_weight(const void* W_hat, aweq_dtype dt, int64_t N, int64_t K, int64_t ldw,
                                 int bits, int group, void* codes, float* step, int32_t* zero,
                                 int32_t* rowsum_w, void* ws, size_t ws_bytes,
                                 uint32_t* status, void* stream)
{
    if (!W_hat || !codes || !step || !zero) return AWEQ_ERR_NULL;
    if (dt != AWEQ_F32 && dt != AWEQ_F16) return AWEQ_ERR_DTYPE;
    if (bits != 8 && bits != 4 && bits != 3) return AWEQ_ERR_BITS;
    if (N <= 0 || K <= 0 || ldw < K || (K % 8) != 0) return AWEQ_ERR_SHAPE;
    if (N > 0x7fffffffll) return AWEQ_ERR_SHAPE;
    if (bits == 3 && (K % 32) != 0) return AWEQ_ERR_ALIGN;
    int levels = -1;
    if (group > 0) {
        for (int l = 0; l <= 6; ++l)
            if (group == (8 << l)) levels = l;
        if (levels < 0 || (K % group) != 0) return AWEQ_ERR_GROUP;
        if (rowsum_w) return AWEQ_ERR_GROUP;  // row sums are defined for per-row / per-tensor int8 only
        if (N > 65535) return AWEQ_ERR_SHAPE;  // rows ride on the grid's y dimension
    } else if (group < -1) {
        return AWEQ_ERR_GROUP;
    } else if (K > (int64_t)kQwBlock * 8 * kQwMaxUnits) {
        return AWEQ_ERR_SHAPE;  // a row must fit the block's registers
    }
    if (!aligned16(W_hat) || ((size_t)ldw * dtype_size(dt)) % 16 != 0 || !aligned16(codes)) return AWEQ_ERR_ALIGN;
    if (group == -1 && (!ws || ws_bytes < 2 * sizeof(uint32_t))) return AWEQ_ERR_WORKSPACE;

    hipStream_t st = as_stream(stream);
    uint8_t* cb = reinterpret_cast<uint8_t*>(codes);
    const bool f16 = dt == AWEQ_F16;
    if (group == -1) {
        uint32_t* keys = reinterpret_cast<uint32_t*>(ws);
        tensor_minmax_init<<<1, 1, 0, st>>>(keys);
        const unsigned g = (unsigned)(N < 2048 ? N : 2048);
        if (f16) tensor_minmax<true><<<g, kQwBlock, 0, st>>>(W_hat, N, K, ldw, keys);
        else tensor_minmax<false><<<g, kQwBlock, 0, st>>>(W_hat, N, K, ldw, keys);
        tensor_qparams<<<1, 1, 0, st>>>(keys, bits, step, zero, status);
    }
#define AWEQ_DISPATCH(F, B)                                                                            \
    if (group > 0) launch_group<F, B>(levels, W_hat, N, K, ldw, cb, step, zero, status, st);           \
    else if (group == -1) launch_row<F, B, true, false>(W_hat, N, K, ldw, cb, step, zero, rowsum_w, status, st);      \
    else launch_row<F, B, false, false>(W_hat, N, K, ldw, cb, step, zero, rowsum_w, status, st);
    if (f16) {
        if (bits == 8) { AWEQ_DISPATCH(true, 8) } else if (bits == 4) { AWEQ_DISPATCH(true, 4) } else { AWEQ_DISPATCH(true, 3) }
    } else {
        if (bits == 8) { AWEQ_DISPATCH(false, 8) } else if (bits == 4) { AWEQ_DISPATCH(false, 4) } else { AWEQ_DISPATCH(false, 3) }
    }
#undef AWEQ_DISPATCH
    return launch_status();
}

// Fold and quantise in one pass over W (per-row quantizer): what aweq_equalize's fold followed by
// aweq_quant_weight with group = 0 produce, with W read once and W_hat not read back.
extern "C" int aweq_fold_quant_weight(const void* W, aweq_dtype dt, int64_t N, int64_t K, int64_t ldw,
                                      const float* s, void* W_hat, int64_t ldwh, int bits, void* codes, float* step,
                                      int32_t* zero, int32_t* rowsum_w, uint32_t* status, void* stream)
{
    if (!W || !s || !W_hat || !codes || !step || !zero) return AWEQ_ERR_NULL;
    if (dt != AWEQ_F32 && dt != AWEQ_F16) return AWEQ_ERR_DTYPE;
    if (bits != 8 && bits != 4 && bits != 3) return AWEQ_ERR_BITS;
    if (N <= 0 || N > 0x7fffffffll || K <= 0 || ldw < K || ldwh < K || (K % 8) != 0) return AWEQ_ERR_SHAPE;
    if (K > (int64_t)kQwBlock * 8 * kQwMaxUnits) return AWEQ_ERR_SHAPE;  // a row must fit the block's registers
    if (bits == 3 && (K % 32) != 0) return AWEQ_ERR_ALIGN;
    if (bits != 8 && rowsum_w) return AWEQ_ERR_BITS;
    if (!aligned16(W) || !aligned16(W_hat) || !aligned16(s) || ((size_t)ldw * dtype_size(dt)) % 16 != 0 ||
        ((size_t)ldwh * dtype_size(dt)) % 16 != 0 || !aligned16(codes))
        return AWEQ_ERR_ALIGN;
    hipStream_t st = as_stream(stream);
    uint8_t* cb = reinterpret_cast<uint8_t*>(codes);
#define AWEQ_FQ(F, B) launch_row<F, B, false, true>(W, N, K, ldw, cb, step, zero, rowsum_w, status, st, s, W_hat, ldwh)
    if (dt == AWEQ_F16) { if (bits == 8) AWEQ_FQ(true, 8); else if (bits == 4) AWEQ_FQ(true, 4); else AWEQ_FQ(true, 3); }
    else { if (bits == 8) AWEQ_FQ(false, 8); else if (bits == 4) AWEQ_FQ(false, 4); else AWEQ_FQ(false, 3); }
#undef AWEQ_FQ
    return launch_status();
}
