// Eq. 10 on one channel, and the range of the equalised activation: shared by the equalization entry point and the calibration of a
// whole layer.
#pragma once
#include "common.hpp"

namespace aweq {

// s of a channel from the extremes of its activations (x0, x1) and weights (w0, w1)
__device__ __forceinline__ float channel_scale(float x0, float x1, float w0, float w1, int enable_awe, uint32_t& st)
{
    // the per-channel quantity the scale balances: the channel range (Eq. 10), or - the definition the
    // method replaces (Sec. 1, Sec. 3.2) - the channel's largest magnitude
    const float r_x = enable_awe == AWEQ_SCALE_ABSMAX ? fmaxf(fabsf(x0), fabsf(x1)) : x1 - x0;
    const float r_w = enable_awe == AWEQ_SCALE_ABSMAX ? fmaxf(fabsf(w0), fabsf(w1)) : w1 - w0;
    float sk = 1.0f;
    if (enable_awe) {
        if (!(r_x >= 1e-5f) || !(r_w >= 1e-5f)) {
            st |= AWEQ_ST_SCALEGUARD;
        } else {
            const double rx = (double)r_x, rw = (double)r_w;
            sk = (float)(sqrt(rx * rw) / rw);
            if (sk < 1e-4f) { sk = 1e-4f; st |= AWEQ_ST_SCALEGUARD; }
            if (sk > 1e4f) { sk = 1e4f; st |= AWEQ_ST_SCALEGUARD; }
        }
    }
    return sk;
}

// The range over all channels that a calibration's merge kernel leaves in pieces, and where the quantities derived from it go.  The
// pieces are min / max per block of channels: of the activations, of the weights, of the equalised activations ([6][blocks]).
constexpr int kRangeCols = 32;   // channels behind a piece
struct RangeParts {
    const float* ext;
    int blocks;
    float* xhat_range;
    float* act_step;
    int32_t* act_zero;
};

// Minimum of rows 2 `pair` and maximum of rows 2 `pair` + 1 of the pieces; every thread of a block of NT calls it and gets both.
// slot: 2 NT / 64 floats (a barrier has to lie between two uses)
template <int NT>
__device__ __forceinline__ float2 parts_extremes(const float* ext, int blocks, int pair, float* slot)
{
    constexpr int NW = NT / kWave;
    float lo = INFINITY, hi = -INFINITY;
    for (int j = threadIdx.x; j < blocks; j += NT) {
        lo = fminf(lo, ext[(2 * pair) * blocks + j]);
        hi = fmaxf(hi, ext[(2 * pair + 1) * blocks + j]);
    }
    lo = wave_allreduce(lo, OpMin());
    hi = wave_allreduce(hi, OpMax());
    if constexpr (NW > 1) {
        const int w = threadIdx.x / kWave;
        if ((threadIdx.x & (kWave - 1)) == 0) { slot[2 * w] = lo; slot[2 * w + 1] = hi; }
        __syncthreads();
#pragma unroll
        for (int i = 0; i < NW; ++i) { lo = fminf(lo, slot[2 * i]); hi = fmaxf(hi, slot[2 * i + 1]); }
    }
    return make_float2(lo, hi);
}

// W_hat = W s (equalize.hip): what the launch asks of its arguments, and the launch
int check_fold_args(const void* W, const void* W_hat, aweq_dtype dt, int64_t N, int64_t K, int64_t ldw, int64_t ldwh);
void launch_fold(const void* W, void* W_hat, aweq_dtype dt, int64_t N, int64_t K, int64_t ldw, int64_t ldwh, const float* s, hipStream_t st);

}  // namespace aweq
