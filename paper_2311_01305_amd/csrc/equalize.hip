// Stage 2: equalization factors (Sec. 3.2, Eq. 10) and the fold of Eq. 3 (Sec. 3.1).
#include "equalize.hpp"

namespace aweq {

// K-vector work: s, inv_s, equalised activation mean, optional prev_scale *= inv_s; and, if `range` is set (one block
// only: it is over all channels and the call has no scratch memory), the equalised activation range with the static
// int8 activation quantizer (Eq. 2 on the range of X_hat).  Bound by the round trips of a block's loads, so a thread of
// the one block requests kScaleBatch channels before it uses the first, and then by its fp64 square roots and divisions: 1 us
// per 1024 channels.  Up to kOneBlockK channels one block does everything, and up to kOneBlockRangeK where the range is asked
// for, which costs several blocks a second launch; beyond, a block per 1024 channels (a thread has one channel then) and
// a launch of equalize_range (us, back to back, one block / two launches: K = 4104 6.4 / 9.0, 5120 7.3 / 9.0, 6144 8.1 / 9.3,
// 7168 8.7 / 9.3, 8192 9.4 / 9.2, 11008 11.9 / 9.0; without the range 4608 6.4 / 6.0, 8192 9.3 / 5.9).  equalize_range reads xmin and xmax again, so a
// call whose vectors replace them stays with one block, which has read a channel's statistics before it writes the channel.
constexpr int kScaleBatch = 4;
constexpr int kScaleBlock = 1024;
constexpr int64_t kOneBlockK = 4096, kOneBlockRangeK = 7168;

// extremes of the equalised activation -> its range and quantizer (every thread of the one block calls it)
__device__ __forceinline__ void finish_range(float lo, float hi, float* slot, float* xhat_range, float* act_step,
                                             int32_t* act_zero, uint32_t& st)
{
    lo = block_allreduce<kScaleBlock / kWave>(lo, OpMin(), slot);
    hi = block_allreduce<kScaleBlock / kWave>(hi, OpMax(), slot);
    if (threadIdx.x == 0) {
        if (xhat_range) { xhat_range[0] = lo; xhat_range[1] = hi; }
        if (act_step && act_zero) {
            float sp; int z;
            qparams(lo, hi, 8, sp, z, st);
            *act_step = sp;
            *act_zero = z;
        }
    }
}

__global__ __launch_bounds__(kScaleBlock) void equalize_scales(
    const float* __restrict__ xmin, const float* __restrict__ xmax, const double* __restrict__ xsum,
    uint64_t count, const float* __restrict__ wmin, const float* __restrict__ wmax, int64_t K,
    int enable_awe, float* __restrict__ s, float* __restrict__ inv_s, float* __restrict__ prev_scale,
    float* __restrict__ xhat_range, float* __restrict__ mu_xhat, float* __restrict__ act_step,
    int32_t* __restrict__ act_zero, uint32_t* status, int range)
{
    __shared__ float slot[kScaleBlock / kWave];
    uint32_t st = 0;
    float lo = INFINITY, hi = -INFINITY;
    const int64_t stride = (int64_t)kScaleBlock * gridDim.x;
    for (int64_t k0 = (int64_t)blockIdx.x * kScaleBlock + threadIdx.x; k0 < K; k0 += kScaleBatch * stride) {
        float x0[kScaleBatch], x1[kScaleBatch], w0[kScaleBatch], w1[kScaleBatch];
        double xs[kScaleBatch];
#pragma unroll
        for (int i = 0; i < kScaleBatch; ++i) {
            const int64_t k = min(k0 + i * stride, K - 1);   // (past the end: the last channel again, not used)
            x0[i] = xmin[k]; x1[i] = xmax[k]; w0[i] = wmin[k]; w1[i] = wmax[k];
            xs[i] = mu_xhat ? xsum[k] : 0.0;
        }
#pragma unroll
        for (int i = 0; i < kScaleBatch; ++i) {
            const int64_t k = k0 + i * stride;
            if (k >= K) break;
            const float sk = channel_scale(x0[i], x1[i], w0[i], w1[i], enable_awe, st);
            const float is = 1.0f / sk;
            s[k] = sk;
            inv_s[k] = is;
            if (prev_scale) prev_scale[k] = prev_scale[k] * is;
            if (mu_xhat) mu_xhat[k] = (float)((xs[i] / (double)count) * (double)is);
            // a correctly rounded multiply by a positive constant is monotone, so the extremes of
            // the equalised column are the scaled extremes of the column
            lo = fminf(lo, x0[i] * is);
            hi = fmaxf(hi, x1[i] * is);
        }
    }
    if (range) finish_range(lo, hi, slot, xhat_range, act_step, act_zero, st);
    raise_status(status, st);
}

__global__ __launch_bounds__(kScaleBlock) void equalize_range(
    const float* __restrict__ xmin, const float* __restrict__ xmax, const float* __restrict__ inv_s, int64_t K,
    float* __restrict__ xhat_range, float* __restrict__ act_step, int32_t* __restrict__ act_zero, uint32_t* status)
{
    __shared__ float slot[kScaleBlock / kWave];
    uint32_t st = 0;
    float lo = INFINITY, hi = -INFINITY;
    for (int64_t k0 = threadIdx.x; k0 < K; k0 += 12 * kScaleBlock) {
        float x0[12], x1[12], is[12];
#pragma unroll
        for (int i = 0; i < 12; ++i) {
            const int64_t k = min(k0 + i * kScaleBlock, K - 1);   // (past the end: the last channel again)
            x0[i] = xmin[k]; x1[i] = xmax[k]; is[i] = inv_s[k];
        }
#pragma unroll
        for (int i = 0; i < 12; ++i) {
            lo = fminf(lo, x0[i] * is[i]);
            hi = fmaxf(hi, x1[i] * is[i]);
        }
    }
    finish_range(lo, hi, slot, xhat_range, act_step, act_zero, st);
    raise_status(status, st);
}

// W_hat[n,k] = W[n,k] * s[k].  Threads own 8 (binary16) or 4 (binary32) columns and walk
// down the rows of their slice, so s stays in registers.
// LAST: the last read of W, non-temporal (rule and figures at the launch)
template <bool F16, bool LAST>
__global__ __launch_bounds__(256) void fold_weight(const void* __restrict__ Wv, void* __restrict__ Ov,
                                                   int64_t N, int64_t K, int64_t ldw, int64_t ldwh,
                                                   const float* __restrict__ s, int64_t rows_per_block)
{
    constexpr int E = F16 ? 8 : 4;
    const int64_t col = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) * E;
    if (col >= K) return;
    float sc[E];
#pragma unroll
    for (int i = 0; i < E; ++i) sc[i] = s[col + i];
    const int64_t n0 = (int64_t)blockIdx.y * rows_per_block;
    const int64_t n1 = min(N, n0 + rows_per_block);
    for (int64_t n = n0; n < n1; ++n) {
        if constexpr (F16) {
            const _Float16* W = reinterpret_cast<const _Float16*>(Wv);
            _Float16* O = reinterpret_cast<_Float16*>(Ov);
            typedef int v4i_ __attribute__((ext_vector_type(4)));
            const v4i_* const q = reinterpret_cast<const v4i_*>(W + n * ldw + col);
            const Half8 v = __builtin_bit_cast(Half8, LAST ? __builtin_nontemporal_load(q) : *q);
            Half8 o;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                float2 f = h2f2(v.h[i]);
                f.x = rounded_f32(f.x * sc[2 * i]);
                f.y = rounded_f32(f.y * sc[2 * i + 1]);
                o.h[i] = f16x2{(_Float16)f.x, (_Float16)f.y};
            }
            *reinterpret_cast<Half8*>(O + n * ldwh + col) = o;
        } else {
            const float* W = reinterpret_cast<const float*>(Wv);
            float* O = reinterpret_cast<float*>(Ov);
            Float4 v = *reinterpret_cast<const Float4*>(W + n * ldw + col);
#pragma unroll
            for (int i = 0; i < 4; ++i) v.f[i] = v.f[i] * sc[i];
            *reinterpret_cast<Float4*>(O + n * ldwh + col) = v;
        }
    }
}

int check_fold_args(const void* W, const void* W_hat, aweq_dtype dt, int64_t N, int64_t K, int64_t ldw, int64_t ldwh)
{
    if (!W || !W_hat) return AWEQ_ERR_NULL;
    if (dt != AWEQ_F32 && dt != AWEQ_F16) return AWEQ_ERR_DTYPE;
    if (N <= 0 || ldw < K || ldwh < K) return AWEQ_ERR_SHAPE;
    if (!aligned16(W) || !aligned16(W_hat) || ((size_t)ldw * dtype_size(dt)) % 16 != 0 || ((size_t)ldwh * dtype_size(dt)) % 16 != 0)
        return AWEQ_ERR_ALIGN;
    return AWEQ_OK;
}

// W_hat = W s on checked arguments
void launch_fold(const void* W, void* W_hat, aweq_dtype dt, int64_t N, int64_t K, int64_t ldw, int64_t ldwh, const float* s, hipStream_t st)
{
    const int E = dt == AWEQ_F16 ? 8 : 4;
    const unsigned gx = (unsigned)cdiv(K, 256 * E);
    int64_t slices = cdiv(4096, gx);
    if (slices > N) slices = N;
    const int64_t rpb = cdiv(N, slices);
    dim3 grid(gx, (unsigned)cdiv(N, rpb));
    // binary16: W is not read again, the folded weight and its codes are: non-temporal, where rows are whole 128-byte lines (after
    // the statistics of W, us, plain -> non-temporal: 4096 x 11008 60.3 -> 55.1, 11008 x 4096 61.4 -> 57.5).  A line that two rows
    // share would be fetched twice (14796 x 2360 58.3 -> 61.4, 8500 x 3224 46.6 -> 49.5)
    const bool lines = reinterpret_cast<uintptr_t>(W) % 128 == 0 && (ldw * 2) % 128 == 0;
    if (dt == AWEQ_F16 && lines)
        fold_weight<true, true><<<grid, 256, 0, st>>>(W, W_hat, N, K, ldw, ldwh, s, rpb);
    else if (dt == AWEQ_F16)
        fold_weight<true, false><<<grid, 256, 0, st>>>(W, W_hat, N, K, ldw, ldwh, s, rpb);
    else
        fold_weight<false, false><<<grid, 256, 0, st>>>(W, W_hat, N, K, ldw, ldwh, s, rpb);
}

}  // namespace aweq

using namespace aweq;

extern "C" int aweq_equalize(const float* xmin, const float* xmax, const double* xsum, uint64_t count,
                             const float* wmin, const float* wmax, int64_t K, int enable_awe,
                             float* s, float* inv_s,
                             const void* W, void* W_hat, aweq_dtype dt, int64_t N, int64_t ldw, int64_t ldwh,
                             float* prev_scale, float* xhat_range, float* mu_xhat,
                             float* act_step, int32_t* act_zero,
                             uint32_t* status, void* stream)
{
    if (!xmin || !xmax || !wmin || !wmax || !s || !inv_s) return AWEQ_ERR_NULL;
    if (mu_xhat && !xsum) return AWEQ_ERR_NULL;
    if ((act_step == nullptr) != (act_zero == nullptr)) return AWEQ_ERR_NULL;
    if (K <= 0 || (K % 8) != 0) return AWEQ_ERR_SHAPE;
    if (enable_awe < 0 || enable_awe > AWEQ_SCALE_ABSMAX) return AWEQ_ERR_SHAPE;
    if (mu_xhat && count == 0) return AWEQ_ERR_SHAPE;
    if (W) {
        const int rc = check_fold_args(W, W_hat, dt, N, K, ldw, ldwh);
        if (rc != AWEQ_OK) return rc;
    }
    hipStream_t st = as_stream(stream);
    const bool range = xhat_range || act_step;
    const bool one = K <= (range ? kOneBlockRangeK : kOneBlockK) ||
                     overlap({{s, K * 4}, {inv_s, K * 4}, {mu_xhat, K * 4}, {prev_scale, K * 4}}, {{xmin, K * 4}, {xmax, K * 4}});
    equalize_scales<<<one ? 1u : (unsigned)cdiv(K, kScaleBlock), kScaleBlock, 0, st>>>(
        xmin, xmax, xsum, count, wmin, wmax, K, enable_awe, s, inv_s, prev_scale, xhat_range, mu_xhat, act_step, act_zero, status, one);
    if (!one && range)
        equalize_range<<<1, kScaleBlock, 0, st>>>(xmin, xmax, inv_s, K, xhat_range, act_step, act_zero, status);
    if (W) launch_fold(W, W_hat, dt, N, K, ldw, ldwh, s, st);
    return launch_status();
}
