// Reductions of several rows' values over a wavefront (or groups of lanes) at once.  Instead of an all-reduce for every row, the first
// two levels hand each lane of a quad the rows it keeps: lane l ends with the total of row l % ROWS, over the lanes that hold it, for
// less than half the instructions of ROWS all-reductions.  Every lane of the wavefront (of the group) has to be active.
#pragma once
#include "common.hpp"

namespace aweq {

// value of the lane that DPP control CTRL names (every lane reads an active one): the compiler merges it into the operation that uses it
template <int CTRL>
__device__ __forceinline__ int dpp_from(int v) { return __builtin_amdgcn_mov_dpp(v, CTRL, 0xf, 0xf, true); }
template <int CTRL>
__device__ __forceinline__ float dpp_from(float v) { return __int_as_float(dpp_from<CTRL>(__float_as_int(v))); }
template <int CTRL>
__device__ __forceinline__ f16x2 dpp_from(f16x2 v) { return __builtin_bit_cast(f16x2, dpp_from<CTRL>(__builtin_bit_cast(int, v))); }
template <int CTRL>
__device__ __forceinline__ double dpp_from(double v) { return __hiloint2double(dpp_from<CTRL>(__double2hiint(v)), dpp_from<CTRL>(__double2loint(v))); }
template <int CTRL>
__device__ __forceinline__ long long dpp_from(long long v)
{
    return ((long long)dpp_from<CTRL>((int)(v >> 32)) << 32) | (unsigned int)dpp_from<CTRL>((int)(v & 0xffffffffll));
}
template <int LVL>
__device__ __forceinline__ f16x2 partner(f16x2 v) { return __builtin_bit_cast(f16x2, partner_bits<LVL>(__builtin_bit_cast(int, v))); }

constexpr int kXor1 = 0xB1, kXor2 = 0x4E, kXor3 = 0x1B, kXor7 = 0x141;   // quad_perm, quad_perm, quad_perm, row_half_mirror
constexpr int kRor4 = 0x124, kRor8 = 0x128;                             // row_ror inside 16 lanes

// LEVELS: over aligned groups of 2^LEVELS lanes (2 at least)
template <int ROWS, int LEVELS, class T, class Op>
__device__ __forceinline__ T reduce_rows(const T (&v)[ROWS], Op op)
{
    static_assert((ROWS == 1 || ROWS == 2 || ROWS == 4) && LEVELS >= 2, "");
    const bool b0 = threadIdx.x & 1, b1 = threadIdx.x & 2;
    T h[ROWS == 4 ? 2 : 1];
    if constexpr (ROWS == 1) h[0] = op(v[0], dpp_from<kXor1>(v[0]));
    else {
#pragma unroll
        for (int i = 0; i < ROWS / 2; ++i) {
            const T keep = b0 ? v[2 * i + 1] : v[2 * i], send = b0 ? v[2 * i] : v[2 * i + 1];
            h[i] = op(keep, dpp_from<kXor1>(send));
        }
    }
    T k;
    if constexpr (ROWS == 4) {
        const T keep = b1 ? h[1] : h[0], send = b1 ? h[0] : h[1];
        k = op(keep, dpp_from<kXor2>(send));
    } else {
        k = op(h[0], dpp_from<kXor2>(h[0]));
    }
    // from here on only lanes with the same l % 4 meet
    if constexpr (LEVELS == 3) k = op(k, dpp_from<kXor3>(dpp_from<kXor7>(k)));   // l ^ 4
    else if constexpr (LEVELS > 3) {
        k = op(k, dpp_from<kRor4>(k));
        k = op(k, dpp_from<kRor8>(k));
    }
    if constexpr (LEVELS > 4) k = op(k, partner<4>(k));
    if constexpr (LEVELS > 5) k = op(k, partner<5>(k));
    return k;
}

struct OpMinH { __device__ f16x2 operator()(f16x2 a, f16x2 b) const { return hmin2(a, b); } };

}  // namespace aweq
