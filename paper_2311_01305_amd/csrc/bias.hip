// Stage 5: quantization bias correction (Sec. 3.3).  delta[n] = mean FP output minus mean
// quantised output over the calibration tokens (Eq. 11); the corrected bias is b + delta.
// By linearity both means contract to K-vectors and integer column sums, so this is a
// GEMV over W_hat (HBM-bound, one read of the weight): fp64 accumulation because delta is a
// small difference of two nearly equal means.
#include "code_digits.hpp"

namespace aweq {

template <bool F16>
__device__ __forceinline__ void load_w8(const void* row, int64_t u, float x[8])
{
    if constexpr (F16) {
        Half8 v = *reinterpret_cast<const Half8*>(reinterpret_cast<const _Float16*>(row) + u * 8);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            float2 f = h2f2(v.h[i]);
            x[2 * i] = f.x;
            x[2 * i + 1] = f.y;
        }
    } else {
        const float* p = reinterpret_cast<const float*>(row) + u * 8;
        Float4 a = *reinterpret_cast<const Float4*>(p), b = *reinterpret_cast<const Float4*>(p + 4);
#pragma unroll
        for (int i = 0; i < 4; ++i) { x[i] = a.f[i]; x[4 + i] = b.f[i]; }
    }
}

// W8A8 (Eq. 11 with the int8 path as the quantised layer):
//   mean_t y[t,n]  = sum_k W_hat[n,k] mu_xhat[k]
//   sum_t  y~[t,n] = Step_x Step_w[n] (colsum_acc[n] - T Z'x rowsum_w[n] - Z'w[n] sum_k colsum_xq[k] + T K Z'x Z'w[n])
// colsum_acc[n] = sum_t acc[t,n] comes from the GEMM, or - by the same linearity, as exact integers -
// from the weight codes: sum_t sum_k xq[t,k] wq[n,k] = sum_k wq[n,k] colsum_xq[k] (wq given, colsum_acc NULL),
// so that calibration does not have to run the forward.
// A block of BLOCK threads takes ROWS output channels at once: mu_xhat and colsum_xq (and their sum over k, which every
// channel needs) are read once per block instead of once per channel.
// The codes meet colsum_xq in 8-bit pieces: a column sum below 2^30 is four signed digits of base 256, and a dot product
// instruction multiplies four codes with four digits of equal weight (one instruction per code; 64-bit products took
// about 15 and bound the kernel).  The four int32 sums of a row grow by at most 2^17 per unit (8 products of at most 2^14), so
// a thread's 2^14 - 1 units are the most that cannot overflow.  Larger column sums and longer rows take the 64-bit products.
// SUMS: compiled for calls that bring colsum_acc, without the registers of the digits.
constexpr int64_t kDigitUnits = (1 << 14) - 1;   // units per thread
template <bool F16, bool SUMS, int BLOCK, int ROWS>
__global__ __launch_bounds__(BLOCK) void bias_w8a8_kernel(
    const void* __restrict__ W_hat, int64_t N, int64_t K, int64_t ldw, const float* __restrict__ mu_xhat, uint64_t count,
    const long long* __restrict__ colsum_acc, const long long* __restrict__ colsum_xq,
    const int32_t* __restrict__ rowsum_w, const float* __restrict__ act_step, const int32_t* __restrict__ act_zero,
    const float* __restrict__ step_w, const int32_t* __restrict__ zero_w, const float* __restrict__ bias_in,
    float* __restrict__ delta, float* __restrict__ bias_out, int enable_bc, const int8_t* __restrict__ codes,
    int w_per_tensor)
{
    const int8_t* const __restrict__ wq = SUMS ? nullptr : codes;
    constexpr int kWaves = BLOCK / kWave;
    __shared__ double slot_d[kWaves][ROWS];
    __shared__ long long slot_l[kWaves][ROWS + 1];
    const int64_t n0 = (int64_t)blockIdx.x * ROWS;
    const int rows = (int)min((int64_t)ROWS, N - n0);
    double acc[ROWS];
    long long ca[ROWS];
    int cd[ROWS][4];
#pragma unroll
    for (int r = 0; r < ROWS; ++r) {
        acc[r] = 0.0;
        ca[r] = 0;
#pragma unroll
        for (int j = 0; j < 4; ++j) cd[r][j] = 0;
    }
    long long tot = 0;
    const bool digits = K / 8 <= kDigitUnits * BLOCK;
    for (int64_t u = threadIdx.x; u < K / 8; u += BLOCK) {
        float w[ROWS][8];
        uint2 v[ROWS];
#pragma unroll
        for (int r = 0; r < ROWS; ++r) {   // (past the edge: the last row again, its results are not stored)
            const int64_t n = n0 + min(r, rows - 1);
            load_w8<F16>(reinterpret_cast<const char*>(W_hat) + (size_t)n * ldw * (F16 ? 2 : 4), u, w[r]);
            // unit u of row n in the K-panel layout: panel u / 8, bytes 8 (u % 8) ..
            if (wq) v[r] = *reinterpret_cast<const uint2*>(wq + ((u >> 3) * N + n) * kPanel + (u & 7) * 8);
        }
        const Float4 m0 = *reinterpret_cast<const Float4*>(mu_xhat + u * 8);
        const Float4 m1 = *reinterpret_cast<const Float4*>(mu_xhat + u * 8 + 4);
        long long cx[8];
        bool small = digits;
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            cx[i] = colsum_xq[u * 8 + i];
            tot += cx[i];
            small = small && cx[i] < (1ll << 30) && cx[i] > -(1ll << 30);
        }
#pragma unroll
        for (int r = 0; r < ROWS; ++r)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                acc[r] = __builtin_fma((double)w[r][i], (double)m0.f[i], acc[r]);
                acc[r] = __builtin_fma((double)w[r][4 + i], (double)m1.f[i], acc[r]);
            }
        if (wq && small) {
            uint32_t d[2][4];
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const int c4[4] = {(int)cx[4 * h], (int)cx[4 * h + 1], (int)cx[4 * h + 2], (int)cx[4 * h + 3]};
                pack_digits(c4, d[h]);
            }
#pragma unroll
            for (int r = 0; r < ROWS; ++r)
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    cd[r][j] = __builtin_amdgcn_sdot4((int)v[r].x, (int)d[0][j], cd[r][j], false);
                    cd[r][j] = __builtin_amdgcn_sdot4((int)v[r].y, (int)d[1][j], cd[r][j], false);
                }
        } else if (wq) {
#pragma unroll
            for (int r = 0; r < ROWS; ++r)
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    ca[r] += (long long)(int8_t)((v[r].x >> (8 * i)) & 0xff) * cx[i];
                    ca[r] += (long long)(int8_t)((v[r].y >> (8 * i)) & 0xff) * cx[4 + i];
                }
        }
    }
    const int wave = threadIdx.x / kWave;
#pragma unroll
    for (int r = 0; r < ROWS; ++r) {
        const double a = wave_allreduce(acc[r], OpAdd());
        if (threadIdx.x % kWave == 0) slot_d[wave][r] = a;
        if (wq) {
            const long long c = wave_allreduce(ca[r] + digits_value(cd[r]), OpAdd());
            if (threadIdx.x % kWave == 0) slot_l[wave][r] = c;
        }
    }
    tot = wave_allreduce(tot, OpAdd());
    if (threadIdx.x % kWave == 0) slot_l[wave][ROWS] = tot;
    __syncthreads();
    if ((int)threadIdx.x >= rows) return;
    const int r = threadIdx.x;
    const int64_t n = n0 + r;
    double a_r = 0.0;
    long long c_r = 0;
    tot = 0;
#pragma unroll
    for (int w = 0; w < kWaves; ++w) {
        a_r += slot_d[w][r];
        if (wq) c_r += slot_l[w][r];
        tot += slot_l[w][ROWS];
    }
    const int64_t pi = w_per_tensor ? 0 : n;   // one (Step, Z) for the tensor, or one per output channel
    const double d = int8_delta(a_r, wq ? c_r : colsum_acc[n], rowsum_w[n], tot, count, K, *act_step, *act_zero, step_w[pi], zero_w[pi]);
    delta[n] = (float)d;
    bias_out[n] = (float)((bias_in ? (double)bias_in[n] : 0.0) + (enable_bc ? d : 0.0));
}

// Weight-only (Eq. 12-15): E[y~ - y] = eps E[x], eps = W~ - W_hat; delta = -eps mu_xhat.
// As above a block takes ROWS output channels, so that mu_xhat and the group of a unit are found once for all of them.
template <bool F16, int BITS, int BLOCK, int ROWS>
__global__ __launch_bounds__(BLOCK) void bias_wonly_kernel(
    const void* __restrict__ W_hat, int64_t N, int64_t K, int64_t ldw, const float* __restrict__ mu_xhat,
    const uint8_t* __restrict__ codes, int64_t group, const float* __restrict__ step_w,
    const int32_t* __restrict__ zero_w, const float* __restrict__ bias_in, float* __restrict__ delta,
    float* __restrict__ bias_out, int enable_bc)
{
    constexpr int kWaves = BLOCK / kWave;
    __shared__ double slot_d[kWaves][ROWS];
    const int64_t n0 = (int64_t)blockIdx.x * ROWS;
    const int rows = (int)min((int64_t)ROWS, N - n0);
    const int64_t g = group > 0 ? group : K;
    const int64_t ng = K / g;
    double acc[ROWS];
#pragma unroll
    for (int r = 0; r < ROWS; ++r) acc[r] = 0.0;
    for (int64_t u = threadIdx.x; u < K / 8; u += BLOCK) {
        // the 8 values of a unit share one group (group sizes are multiples of 8)
        const int64_t gi = K < (1ll << 31) ? (int64_t)((uint32_t)(u * 8) / (uint32_t)g) : (u * 8) / g;
        float w[ROWS][8], sp[ROWS];
        int z[ROWS];
        uint2 v[ROWS];   // the unit's codes as stored: 8, 4 or 3 bytes
#pragma unroll
        for (int r = 0; r < ROWS; ++r) {   // (past the edge: the last row again, its result is not stored)
            const int64_t n = n0 + min(r, rows - 1);
            load_w8<F16>(reinterpret_cast<const char*>(W_hat) + (size_t)n * ldw * (F16 ? 2 : 4), u, w[r]);
            const uint8_t* const crow = codes + (size_t)n * (K * BITS / 8);
            if constexpr (BITS == 8) {
                // per-row / per-tensor 8-bit codes are stored in the GEMM's K-panel layout
                v[r] = group > 0 ? *reinterpret_cast<const uint2*>(crow + u * 8)
                                 : *reinterpret_cast<const uint2*>(codes + ((u >> 3) * N + n) * kPanel + (u & 7) * 8);
            } else if constexpr (BITS == 4) {
                v[r].x = *reinterpret_cast<const uint32_t*>(crow + u * 4);
            } else if constexpr (ROWS < 4) {
                // the unit's 24 bits in one load of 4 bytes, of which a quad's last unit has the upper three
                const int last = (u & 3) == 3;
                uint32_t x;
                __builtin_memcpy(&x, crow + u * 3 - last, 4);
                v[r].x = x >> (8 * last);
            } else {
                // (two aligned loads where four channels make up for them: binary16 8192 x 22016 103 -> 85 us)
                // 24 bits of the 12 bytes four units share (K % 32 == 0: they start on 4-byte boundaries)
                const uint32_t* const q = reinterpret_cast<const uint32_t*>(crow + (u >> 2) * 12);
                const int d = (int)(u & 3);
                v[r].x = __builtin_amdgcn_alignbit(q[min(d, 2)], q[max(d - 1, 0)], (32 - 8 * d) & 31);
            }
            const int64_t pi = group < 0 ? 0 : n * ng + gi;
            sp[r] = step_w[pi];
            z[r] = zero_w[pi];
        }
        const Float4 m0 = *reinterpret_cast<const Float4*>(mu_xhat + u * 8);
        const Float4 m1 = *reinterpret_cast<const Float4*>(mu_xhat + u * 8 + 4);
#pragma unroll
        for (int r = 0; r < ROWS; ++r)
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                const int c = BITS == 8 ? (int)(int8_t)(((i < 4 ? v[r].x : v[r].y) >> (8 * (i & 3))) & 0xff) + 128
                                        : (int)((v[r].x >> (BITS * i)) & ((1u << BITS) - 1u));
                const float wt = (float)(c - z[r]) * sp[r];
                const double eps = (double)wt - (double)w[r][i];
                acc[r] = __builtin_fma(eps, (double)(i < 4 ? m0.f[i] : m1.f[i - 4]), acc[r]);
            }
    }
#pragma unroll
    for (int r = 0; r < ROWS; ++r) {
        const double a = wave_allreduce(acc[r], OpAdd());
        if (threadIdx.x % kWave == 0) slot_d[threadIdx.x / kWave][r] = a;
    }
    __syncthreads();
    if ((int)threadIdx.x >= rows) return;
    const int64_t n = n0 + threadIdx.x;
    double a = 0.0;
#pragma unroll
    for (int w = 0; w < kWaves; ++w) a += slot_d[w][threadIdx.x];
    const double d = -a;
    delta[n] = (float)d;
    bias_out[n] = (float)((bias_in ? (double)bias_in[n] : 0.0) + (enable_bc ? d : 0.0));
}

}  // namespace aweq

using namespace aweq;

extern "C" int aweq_bias_correct(int mode, const void* W_hat, aweq_dtype dt, int64_t N, int64_t K, int64_t ldw,
                                 const float* mu_xhat, uint64_t count,
                                 const int64_t* colsum_acc, const int64_t* colsum_xq, const int32_t* rowsum_w,
                                 const float* act_step, const int32_t* act_zero,
                                 const void* codes, int bits, int group,
                                 const float* step_w, const int32_t* zero_w,
                                 const float* bias_in, float* delta, float* bias_out, int enable_bc,
                                 uint32_t* status, void* stream)
{
    (void)status;   // this stage meets no numeric condition it would have to report
    if (!W_hat || !mu_xhat || !step_w || !zero_w || !delta || !bias_out) return AWEQ_ERR_NULL;
    if (dt != AWEQ_F32 && dt != AWEQ_F16) return AWEQ_ERR_DTYPE;
    if (N <= 0 || N > 0x7fffffffll || K <= 0 || ldw < K || (K % 8) != 0) return AWEQ_ERR_SHAPE;
    if (!aligned16(W_hat) || ((size_t)ldw * dtype_size(dt)) % 16 != 0 || !aligned16(mu_xhat)) return AWEQ_ERR_ALIGN;
    hipStream_t st = as_stream(stream);
    const bool f16 = dt == AWEQ_F16;
    if (mode == AWEQ_BIAS_W8A8) {
        if (!colsum_xq || !rowsum_w || !act_step || !act_zero) return AWEQ_ERR_NULL;
        if (!colsum_acc && !codes) return AWEQ_ERR_NULL;
        if (count == 0) return AWEQ_ERR_SHAPE;
        // without the GEMM's column sums they are formed from the 8-bit per-row / per-tensor codes (K-panel layout)
        const int8_t* wq = colsum_acc ? nullptr : reinterpret_cast<const int8_t*>(codes);
        if (wq && (bits != 8 || group > 0)) return AWEQ_ERR_BITS;
        if (group != 0 && group != -1) return AWEQ_ERR_GROUP;   // the int8 path has one scale per output channel or per tensor
        const int pt = group == -1;
        if (wq && !aligned16(wq)) return AWEQ_ERR_ALIGN;
        const long long* ca = reinterpret_cast<const long long*>(colsum_acc);
        const long long* cx = reinterpret_cast<const long long*>(colsum_xq);
#define AWEQ_B8(F, S, BLOCK, ROWS)                                                                                     \
    bias_w8a8_kernel<F, S, BLOCK, ROWS><<<(unsigned)cdiv(N, ROWS), BLOCK, 0, st>>>(                                    \
        W_hat, N, K, ldw, mu_xhat, count, ca, cx, rowsum_w, act_step, act_zero, step_w, zero_w, bias_in, delta, bias_out, enable_bc, wq, pt)
        // us, threads x channels of a block: small blocks, more of them in flight while others reduce (binary16 from the codes
        // 4096 x 11008: 128 x 4 24.2, 256 x 8 27.6, 256 x 4 26.6, 512 x 8 32.6, 64 x 4 33.4; with 64-bit products and a barrier pair per
        // channel 40.8), but a weight that does not fit the memory-side cache wants more of its long rows on their way (128 x 4 ->
        // 256 x 8: from the codes binary16 22016 x 8192 113 -> 100, 8192 x 22016 130 -> 103; with the GEMM's sums binary16 22016 x 8192
        // 79 -> 70, 8192 x 22016 92 -> 74, 12288 x 12288 65 -> 56, binary32 8192 x 22016 145 -> 128), and binary16 with sums, a read of
        // the weight alone, eight channels of its short ones (40000 x 4096 71 -> 65).  The threads of a block decide the order of
        // the sums: they are the same for both sources of the integers, so that delta is.
        const bool beyond = N * K * (int64_t)dtype_size(dt) >= kCacheBytes, large = beyond && K >= 8192;
        if (f16) {
            if (K <= 1024) AWEQ_B8(true, false, 64, 2);
            else if (large && !wq) AWEQ_B8(true, true, 256, 8);
            else if (large) AWEQ_B8(true, false, 256, 8);
            else if (beyond && !wq) AWEQ_B8(true, true, 128, 8);
            else AWEQ_B8(true, false, 128, 4);
        } else {   // (without the digits' registers binary32 is no faster: 8192 x 22016 128 -> 139)
            if (K <= 1024) AWEQ_B8(false, false, 64, 2);
            else if (large) AWEQ_B8(false, false, 256, 8);
            else AWEQ_B8(false, false, 128, 4);
        }
#undef AWEQ_B8
    } else if (mode == AWEQ_BIAS_WEIGHT_ONLY) {
        if (!codes) return AWEQ_ERR_NULL;
        if (bits != 8 && bits != 4 && bits != 3) return AWEQ_ERR_BITS;
        if (group < -1 || (group > 0 && ((group % 8) != 0 || (K % group) != 0))) return AWEQ_ERR_GROUP;
        if (!aligned16(codes)) return AWEQ_ERR_ALIGN;
        if (bits == 3 && (K % 32) != 0) return AWEQ_ERR_ALIGN;
        const uint8_t* cb = reinterpret_cast<const uint8_t*>(codes);
#define AWEQ_BWS(F, B, BLOCK, ROWS)                                                                                    \
    bias_wonly_kernel<F, B, BLOCK, ROWS><<<(unsigned)cdiv(N, ROWS), BLOCK, 0, st>>>(                                    \
        W_hat, N, K, ldw, mu_xhat, cb, group, step_w, zero_w, bias_in, delta, bias_out, enable_bc)
        // Four channels a block where that leaves enough blocks and their values fit the registers, two otherwise (us, 4 -> 2: binary32,
        // whose channel takes eight registers, INT3 4096 x 11008 49.4 -> 30.0, INT4 8192 x 8192 55.7 -> 45.5; binary16 8-bit groups
        // 4096 x 11008 24.1 -> 22.7, INT3 4096 x 11008 21.1 -> 20.4, INT4 1000 x 16384 14.0 -> 9.9; but 8-bit rows 8192 x 22016 105 -> 114)
        const bool four = f16 && N >= 8192 && !(bits == 8 && group > 0);
        // Few channels of long rows are bound by the passes over a row: 512 threads on one channel (us, 256 x 2 -> 512 x 1: binary32
        // INT4 64 x 21632 7.8 -> 5.5, 3664 x 8576 23.5 -> 21.9; binary16 INT3 256 x 17216 6.8 -> 5.6, 1280 x 11008 9.3 -> 8.8, but 2048 x
        // 11008 11.8 -> 12.2; 8-bit rows, whose panels neighbouring channels share, 512 x 13248 7.1 -> 5.8, 1000 x 16384 11.4 -> 12.7;
        // up to K = 8192 the two take the same)
        const bool longrows = K > 8192 && N <= (bits == 8 && group <= 0 ? 512 : f16 ? 1280 : 4096);
#define AWEQ_BW(F, B) do { if (K <= 1024) AWEQ_BWS(F, B, 64, 2); else if (longrows) AWEQ_BWS(F, B, 512, 1); else if (F && four) AWEQ_BWS(F, B, 256, F ? 4 : 2); else AWEQ_BWS(F, B, 256, 2); } while (0)
        if (f16) { if (bits == 8) AWEQ_BW(true, 8); else if (bits == 4) AWEQ_BW(true, 4); else AWEQ_BW(true, 3); }
        else { if (bits == 8) AWEQ_BW(false, 8); else if (bits == 4) AWEQ_BW(false, 4); else AWEQ_BW(false, 3); }
#undef AWEQ_BW
#undef AWEQ_BWS
    } else {
        return AWEQ_ERR_SHAPE;
    }
    return launch_status();
}
