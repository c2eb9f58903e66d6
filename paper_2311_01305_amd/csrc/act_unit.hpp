// Eq. 1 with b = 8 on 8 values of an equalised activation: the inner step of the activation quantizer (whose header explains
// the division-free quotients) and of the few-token int8 GEMM that quantises its own input.
#pragma once
#include "common.hpp"

namespace aweq {

// One unit (8 consecutive columns of one row): packed codes (returned), column / row sums.
// FAST: the division-free quotient; the unsigned code is kept as an (integral) float, packed
// with v_cvt_pk_u8_f32 and turned into the stored signed code by flipping the top bit
// (u - 128 = u ^ 0x80 as a byte).  Column sums accumulate u in fp32 (exact: at most 512 rows
// of values <= 255 per block); the caller subtracts 128 per row afterwards.
// MODE 0: true division; 1: the exact division-free quotient; 2: screened (see the header); 3: screened for binary32
// input, whose quotients have no bound known beforehand: a unit with one beyond 2^22, infinite or NaN is divided.
// SUMS: only the column sums are wanted (no code buffer, no row sums).
template <int MODE, bool SUMS = false>
__device__ __forceinline__ uint2 act_unit(const float x[8], const float is[8], const ActParams& p,
                                          float csf[8], int csi[8], int& rs, float& big, uint32_t& st)
{
    uint32_t w[2] = {0u, 0u};
    if constexpr (MODE == 2 || MODE == 3) {
        const float zf = (float)p.zero;
        float n[8];
        float dmax = 0.0f, largest = 0.0f, bad = 0.0f;
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            // x is a widened binary16 value: a = RN(x inv_s) as one mixed-precision FMA (+0 changes
            // nothing but the sign of a zero, which the quotient's rounding forgets)
            const float a = __builtin_fmaf(x[i], is[i], 0.0f);
            const float q = __builtin_fmaf(a, p.rstep, zf);
            n[i] = rintf(q);
            const float d = fabsf(q - n[i]);
            dmax = fmaxf(dmax, d);
            if constexpr (MODE == 3) {
                largest = fmaxf(largest, fabsf(q));
                bad += d;   // NaN from an infinite or NaN quotient on
            }
        }
        if (MODE == 3 && !(largest < 4194304.0f && bad < 8.0f)) {
#pragma unroll
            for (int i = 0; i < 8; ++i) n[i] = (float)quant_div(x[i] * is[i], p.step, p.zero, 255, st);
        } else if (dmax > p.thr) {
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                const float a = x[i] * is[i];
                float q = a * p.rstep;
                float r = __builtin_fmaf(-p.step, q, a);
                q = __builtin_fmaf(r, p.rstep, q);
                r = __builtin_fmaf(-p.step, q, a);
                q = __builtin_fmaf(r, p.rstep, q);
                n[i] = rintf(q) + zf;   // |rint| < 2^24 here (checked per thread), |Z| <= 4096
            }
        }
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const float u = __builtin_amdgcn_fmed3f(n[i], 0.0f, 255.0f);
            csf[i] += u;
            if constexpr (!SUMS) w[i >> 2] = __builtin_amdgcn_cvt_pk_u8_f32(u, i & 3, w[i >> 2]);
        }
        w[0] ^= 0x80808080u;
        w[1] ^= 0x80808080u;
    } else if constexpr (MODE == 1) {
        const float zf = (float)p.zero;
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const float a = x[i] * is[i];
            float q = a * p.rstep;
            float r = __builtin_fmaf(-p.step, q, a);
            q = __builtin_fmaf(r, p.rstep, q);
            r = __builtin_fmaf(-p.step, q, a);
            q = __builtin_fmaf(r, p.rstep, q);
            const float n = rintf(q);
            big = fmaxf(big, fabsf(n));
            // |Z| < 2^23: n + Z is exact wherever it can land inside [0, 255]
            const float u = __builtin_amdgcn_fmed3f(n + zf, 0.0f, 255.0f);
            csf[i] += u;
            w[i >> 2] = __builtin_amdgcn_cvt_pk_u8_f32(u, i & 3, w[i >> 2]);
        }
        w[0] ^= 0x80808080u;
        w[1] ^= 0x80808080u;
    } else {
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const float a = x[i] * is[i];
            const int c = quant_div(a, p.step, p.zero, 255, st) - 128;
            csi[i] += c;
            w[i >> 2] |= (uint32_t)(c & 0xff) << (8 * (i & 3));
        }
    }
    if constexpr (!SUMS) {
        rs = __builtin_amdgcn_sdot4((int)w[0], 0x01010101, rs, false);
        rs = __builtin_amdgcn_sdot4((int)w[1], 0x01010101, rs, false);
    }
    return make_uint2(w[0], w[1]);
}

// 8 consecutive input values of one row as loaded (binary16: one 16-byte quad), converted to
// fp32 only when they are consumed so that the loads in flight stay cheap in registers
template <bool F16> struct RawUnit;
template <> struct RawUnit<true> {
    Half8 v;
    __device__ __forceinline__ void load(const void* X, int64_t elt)
    {
        typedef int v4i_ __attribute__((ext_vector_type(4)));
        const v4i_ r = __builtin_nontemporal_load(reinterpret_cast<const v4i_*>(reinterpret_cast<const _Float16*>(X) + elt));
        v = __builtin_bit_cast(Half8, r);
    }
    // values that other workgroups read as well (non-temporal, each of them went to memory: one token 4096 x 4096 6.2 us instead of 5.15)
    __device__ __forceinline__ void load_shared(const void* X, int64_t elt)
    {
        v = *reinterpret_cast<const Half8*>(reinterpret_cast<const _Float16*>(X) + elt);
    }
    __device__ __forceinline__ void get(float x[8]) const
    {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            float2 f = h2f2(v.h[i]);
            x[2 * i] = f.x;
            x[2 * i + 1] = f.y;
        }
    }
};
template <> struct RawUnit<false> {
    Float4 a, b;
    __device__ __forceinline__ void load(const void* X, int64_t elt)
    {
        const float* p = reinterpret_cast<const float*>(X) + elt;
        a = *reinterpret_cast<const Float4*>(p);
        b = *reinterpret_cast<const Float4*>(p + 4);
    }
    __device__ __forceinline__ void load_shared(const void* X, int64_t elt) { load(X, elt); }
    __device__ __forceinline__ void get(float x[8]) const
    {
#pragma unroll
        for (int i = 0; i < 4; ++i) { x[i] = a.f[i]; x[4 + i] = b.f[i]; }
    }
};

// Codes of one unit with the quotient its wavefront may take (every lane of it calls this); no column sums
template <bool F16>
__device__ __forceinline__ uint2 act_unit_any(const float x[8], const float is[8], const ActParams& p, int& rs, float& big, uint32_t& st)
{
    bool fast = p.fast;
    float is_max = 0.0f;
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        // the exactness argument needs a y not to overflow: binary16 |x| < 2^16, Step >= 2^-60
        if (!(fabsf(is[i]) < 1.0e12f)) fast = false;
        is_max = fmaxf(is_max, fabsf(is[i]));
    }
    // the screened path does not track the largest quotient: it needs |x inv_s / Step| < 2^24 up front (with a margin)
    const bool screen = __all(fast && p.screen && 65600.0f * is_max * p.rstep < 16777216.0f);
    const bool exact = __all(fast);
    float csf[8] = {};
    int csi[8] = {};
    if (!F16 && p.screen) return act_unit<3>(x, is, p, csf, csi, rs, big, st);
    if (F16 && screen) return act_unit<2>(x, is, p, csf, csi, rs, big, st);
    if (F16 && exact) return act_unit<1>(x, is, p, csf, csi, rs, big, st);
    return act_unit<0>(x, is, p, csf, csi, rs, big, st);
}

}  // namespace aweq
