// Units of 8 consecutive weights of one row and their codes (Eq. 1-2): shared by the weight quantizer and by the pass that folds,
// quantises and corrects the bias in one read of the weight.
//
// Eq. 1's quotient without a division: the screened and the exact quotient of the activation quantizer, per slice where
// their conditions hold (Step's exponent and significand, |Z| <= 4096) and no element of the wavefront is NaN or reaches a
// quotient of 2^23 (nothing overflows then and BIGQUOT cannot occur; a binary32 element so small that a product underflows
// has the code Z either way).  With the division (about 45 operations an element) the kernels were bound by the vector unit.
#pragma once
#include "common.hpp"

namespace aweq {

template <bool F16>
struct Unit;

template <>
struct Unit<true> {
    Half8 raw;
    __device__ __forceinline__ void load(const void* row, int64_t u)
    {
        raw = *reinterpret_cast<const Half8*>(reinterpret_cast<const _Float16*>(row) + u * 8);
    }
    __device__ __forceinline__ void get(float x[8]) const
    {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            float2 f = h2f2(raw.h[i]);
            x[2 * i] = f.x;
            x[2 * i + 1] = f.y;
        }
    }
    // round to binary16 and keep
    __device__ __forceinline__ void set(const float x[8])
    {
#pragma unroll
        for (int i = 0; i < 4; ++i) raw.h[i] = f16x2{(_Float16)x[2 * i], (_Float16)x[2 * i + 1]};
    }
    __device__ __forceinline__ void store(void* row, int64_t u) const
    {
        *reinterpret_cast<Half8*>(reinterpret_cast<_Float16*>(row) + u * 8) = raw;
    }
};

template <>
struct Unit<false> {
    Float4 raw[2];
    __device__ __forceinline__ void load(const void* row, int64_t u)
    {
        const float* p = reinterpret_cast<const float*>(row) + u * 8;
        raw[0] = *reinterpret_cast<const Float4*>(p);
        raw[1] = *reinterpret_cast<const Float4*>(p + 4);
    }
    __device__ __forceinline__ void get(float x[8]) const
    {
#pragma unroll
        for (int i = 0; i < 4; ++i) { x[i] = raw[0].f[i]; x[4 + i] = raw[1].f[i]; }
    }
    __device__ __forceinline__ void set(const float x[8])
    {
#pragma unroll
        for (int i = 0; i < 4; ++i) { raw[0].f[i] = x[i]; raw[1].f[i] = x[4 + i]; }
    }
    __device__ __forceinline__ void store(void* row, int64_t u) const
    {
        float* p = reinterpret_cast<float*>(row) + u * 8;
        *reinterpret_cast<Float4*>(p) = raw[0];
        *reinterpret_cast<Float4*>(p + 4) = raw[1];
    }
};

__device__ __forceinline__ void minmax8(const float x[8], float& lo, float& hi)
{
#pragma unroll
    for (int i = 0; i < 8; ++i) { lo = fminf(lo, x[i]); hi = fmaxf(hi, x[i]); }
}

// Extremes of the elements seen so far (binary16: in pairs), and whether one of them was NaN or infinite
template <bool F16> struct Extremes;
template <>
struct Extremes<true> {
    f16x2 lo = {(_Float16)INFINITY, (_Float16)INFINITY}, hi = {(_Float16)-INFINITY, (_Float16)-INFINITY}, bad = {(_Float16)0.0f, (_Float16)0.0f};
    __device__ __forceinline__ void add(const Unit<true>& u)
    {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            lo = hmin2(lo, u.raw.h[i]);
            hi = hmax2(hi, u.raw.h[i]);
            bad = __builtin_elementwise_fma(u.raw.h[i], f16x2{(_Float16)0.0f, (_Float16)0.0f}, bad);   // 0, or NaN from then on
        }
    }
    __device__ __forceinline__ float min() const { return fminf((float)lo.x, (float)lo.y); }
    __device__ __forceinline__ float max() const { return fmaxf((float)hi.x, (float)hi.y); }
    __device__ __forceinline__ bool finite() const { return bad.x == (_Float16)0.0f && bad.y == (_Float16)0.0f; }
};
template <>
struct Extremes<false> {
    float lo = INFINITY, hi = -INFINITY, bad = 0.0f;
    __device__ __forceinline__ void add(const Unit<false>& u)
    {
        float x[8];
        u.get(x);
        minmax8(x, lo, hi);
#pragma unroll
        for (int i = 0; i < 8; ++i) bad = __builtin_fmaf(x[i], 0.0f, bad);
    }
    __device__ __forceinline__ float min() const { return lo; }
    __device__ __forceinline__ float max() const { return hi; }
    __device__ __forceinline__ bool finite() const { return bad == 0.0f; }
};

// this thread's elements may take the screened quotient (a thread without elements agrees)
template <bool F16>
__device__ __forceinline__ bool may_screen(const Extremes<F16>& ex, const ActParams& p)
{
    const float lo = ex.min(), hi = ex.max();
    return p.screen && ex.finite() && (lo > hi || fmaxf(fabsf(lo), fabsf(hi)) * p.rstep < 8388608.0f);
}

// the codes of one unit as integral floats (8 bits: not clamped yet), for elements that may_screen accepts
template <int BITS>
__device__ __forceinline__ void unit_codes(const float x[8], const ActParams& p, float u[8])
{
    constexpr float qmax = (float)((1 << BITS) - 1);
    const float zf = (float)p.zero;
    float dmax = 0.0f;
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        const float q = __builtin_fmaf(x[i], p.rstep, zf);
        u[i] = rintf(q);
        dmax = fmaxf(dmax, fabsf(q - u[i]));
    }
    if (dmax > p.thr) {
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            float q = x[i] * p.rstep;
            float r = __builtin_fmaf(-p.step, q, x[i]);
            q = __builtin_fmaf(r, p.rstep, q);
            r = __builtin_fmaf(-p.step, q, x[i]);
            q = __builtin_fmaf(r, p.rstep, q);
            u[i] = rintf(q) + zf;
        }
    }
    if constexpr (BITS == 8) return;   // (the conversion to a byte clamps)
#pragma unroll
    for (int i = 0; i < 8; ++i) u[i] = __builtin_amdgcn_fmed3f(u[i], 0.0f, qmax);
}

// The codes of one unit, packed as stored (8 bits: minus 128, in w0 and w1; 4 / 3 bits: in w0).  DIFF: also u - Z of each, the
// factor of Step in the de-quantised weight.  screened: may_screen holds.
template <int BITS, bool DIFF = false>
__device__ __forceinline__ void unit_words(const float x[8], const ActParams& p, bool screened, uint32_t& w0, uint32_t& w1,
                                           uint32_t& st, float* diff = nullptr)
{
    static_assert(BITS != 8 || !DIFF, "8-bit codes are clamped by their conversion only, after the differences");
    constexpr int qmax = (1 << BITS) - 1;
    w0 = 0;
    w1 = 0;
    if (screened) {
        float c[8];
        unit_codes<BITS>(x, p, c);
        if constexpr (DIFF) {
            const float zf = (float)p.zero;
#pragma unroll
            for (int i = 0; i < 8; ++i) diff[i] = c[i] - zf;   // (exact: |Z| <= 4096)
        }
        if constexpr (BITS == 8) {
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                w0 = __builtin_amdgcn_cvt_pk_u8_f32(c[i], i, w0);
                w1 = __builtin_amdgcn_cvt_pk_u8_f32(c[4 + i], i, w1);
            }
            w0 ^= 0x80808080u;
            w1 ^= 0x80808080u;
        } else {   // Horner's rule in binary32: 4 codes of 4 bits, 8 of 3 bits are below 2^24
            constexpr float base = (float)(1 << BITS);
            float a = c[3], b = c[7];
#pragma unroll
            for (int i = 2; i >= 0; --i) { a = __builtin_fmaf(a, base, c[i]); b = __builtin_fmaf(b, base, c[4 + i]); }
            if constexpr (BITS == 4) w0 = (uint32_t)a | ((uint32_t)b << 16);
            else w0 = (uint32_t)__builtin_fmaf(b, 4096.0f, a);
        }
    } else {
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const int c = quant_div(x[i], p.step, p.zero, qmax, st);
            if constexpr (DIFF) diff[i] = (float)(c - p.zero);
            if constexpr (BITS == 8) (i < 4 ? w0 : w1) |= (uint32_t)((c - 128) & 0xff) << (8 * (i & 3));
            else w0 |= (uint32_t)c << (BITS * i);
        }
    }
}

// Store the codes of unit u of a row whose code bytes start at `row_codes` (bits == 8: the unit sits at row_codes + unit_off, which
// lets the caller pick the layout).  For bits == 3 all four lanes of a quad must call this with consecutive units (u % 4 == lane % 4).
template <int BITS>
__device__ __forceinline__ void store_unit_words(uint32_t w0, uint32_t w1, uint8_t* row_codes, int64_t u, int64_t unit_off = -1)
{
    if constexpr (BITS == 8) {
        *reinterpret_cast<uint2*>(row_codes + (unit_off >= 0 ? unit_off : u * 8)) = make_uint2(w0, w1);
    } else if constexpr (BITS == 4) {
        *reinterpret_cast<uint32_t*>(row_codes + u * 4) = w0;
    } else {
        // 8 codes = 24 bits; four neighbouring lanes hold 96 bits = three dwords
        const uint32_t v0 = (uint32_t)dpp_mov<0x00>((int)w0);  // quad_perm [0,0,0,0]
        const uint32_t v1 = (uint32_t)dpp_mov<0x55>((int)w0);  // [1,1,1,1]
        const uint32_t v2 = (uint32_t)dpp_mov<0xAA>((int)w0);  // [2,2,2,2]
        const uint32_t v3 = (uint32_t)dpp_mov<0xFF>((int)w0);  // [3,3,3,3]
        const int q = threadIdx.x & 3;
        const uint32_t d = q == 0 ? (v0 | (v1 << 24)) : (q == 1 ? ((v1 >> 8) | (v2 << 16)) : ((v2 >> 16) | (v3 << 8)));
        if (q < 3) *reinterpret_cast<uint32_t*>(row_codes + (u >> 2) * 12 + q * 4) = d;
    }
}

// sum of the signed codes of an 8-bit unit
__device__ __forceinline__ int unit_sum(uint32_t w0, uint32_t w1)
{
    return __builtin_amdgcn_sdot4((int)w1, 0x01010101, __builtin_amdgcn_sdot4((int)w0, 0x01010101, 0, false), false);
}

// Quantise one unit and store its codes.  Returns sum (u - 128) (8 bits only).
template <int BITS>
__device__ __forceinline__ int quant_store_unit(const float x[8], const ActParams& p, bool screened, uint8_t* row_codes,
                                                int64_t u, uint32_t& st, int64_t unit_off = -1)
{
    uint32_t w0, w1;
    unit_words<BITS>(x, p, screened, w0, w1, st);
    store_unit_words<BITS>(w0, w1, row_codes, u, unit_off);
    return BITS == 8 ? unit_sum(w0, w1) : 0;
}

}  // namespace aweq
