// Dot products of 8-bit codes with larger integers: an integer below 2^30 in absolute value is four signed digits of base 256, and one
// instruction multiplies four codes with four digits of equal weight.
#pragma once
#include "common.hpp"

namespace aweq {

// digit j of cx[0 .. 3], packed into d[j]: adding 0x808080 carries into the digit above, and flipping the lower digits' top bits
// takes it back out
__device__ __forceinline__ void pack_digits(const int cx[4], uint32_t d[4])
{
    uint32_t b[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) b[i] = ((uint32_t)cx[i] + 0x00808080u) ^ 0x00808080u;
    const uint32_t l01 = __builtin_amdgcn_perm(b[1], b[0], 0x05010400u), l23 = __builtin_amdgcn_perm(b[3], b[2], 0x05010400u);
    const uint32_t h01 = __builtin_amdgcn_perm(b[1], b[0], 0x07030602u), h23 = __builtin_amdgcn_perm(b[3], b[2], 0x07030602u);
    d[0] = __builtin_amdgcn_perm(l23, l01, 0x05040100u);
    d[1] = __builtin_amdgcn_perm(l23, l01, 0x07060302u);
    d[2] = __builtin_amdgcn_perm(h23, h01, 0x05040100u);
    d[3] = __builtin_amdgcn_perm(h23, h01, 0x07060302u);
}

// sum of the four digits' partial dot products
__device__ __forceinline__ long long digits_value(const int cd[4])
{
    return cd[0] + ((long long)cd[1] << 8) + ((long long)cd[2] << 16) + ((long long)cd[3] << 24);
}

// Eq. 11 for one output channel of the int8 path: mean FP output a_fp minus the mean quantised output, from the accumulator's sum over
// the tokens (colsum_acc), the codes' row sum and the total of the activation codes' column sums
__device__ __forceinline__ double int8_delta(double a_fp, long long colsum_acc, long long rowsum, long long tot, uint64_t count, int64_t K,
                                             float act_step, int act_zero, float step_w, int zero_w)
{
    const long long T = (long long)count;
    const long long zx = (long long)act_zero - 128, zw = (long long)zero_w - 128;
    const long long a = colsum_acc - T * zx * rowsum - zw * tot + T * K * zx * zw;
    return a_fp - (double)act_step * (double)step_w * (double)a / (double)T;
}

}  // namespace aweq
