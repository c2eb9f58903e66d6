// De-quantisation of packed 4-bit / 3-bit weight codes to binary16, shared by the weight-only kernels:
// w~_h = RN16((u - Z) RN16(Step)) (Eq. 1 with the weight operand in binary16).
#pragma once
#include "common.hpp"

namespace aweq {
namespace wonly {

typedef int v4i __attribute__((ext_vector_type(4)));

__device__ __forceinline__ f16x2 as_h2(uint32_t u) { return __builtin_bit_cast(f16x2, u); }
__device__ __forceinline__ uint32_t as_u32(f16x2 h) { return __builtin_bit_cast(uint32_t, h); }

// 32 consecutive codes of one row as loaded: 16 (INT4) or 12 (INT3) bytes
template <int BITS> struct RawCodes { uint32_t w[BITS == 4 ? 4 : 3]; };

template <int BITS>
__device__ __forceinline__ RawCodes<BITS> load_codes(const uint8_t* p)
{
    RawCodes<BITS> rc;
    if constexpr (BITS == 4) {
        const v4i w = *reinterpret_cast<const v4i*>(p);
        rc.w[0] = (uint32_t)w[0]; rc.w[1] = (uint32_t)w[1]; rc.w[2] = (uint32_t)w[2]; rc.w[3] = (uint32_t)w[3];
    } else {
        // rows of 3-bit codes start on 4-byte boundaries only
        const uint32_t* p32 = reinterpret_cast<const uint32_t*>(p);
        rc.w[0] = p32[0]; rc.w[1] = p32[1]; rc.w[2] = p32[2];
    }
    return rc;
}

// Step and Z of one slice, ready for dequant8.  A code field at bit b of a binary16 significand whose
// exponent makes that bit worth 1 reads as 2^(10 - b) + u, so subtracting 2^(10 - b) + Z leaves u - Z
// (exact: both are integers below 2048), and no shift is needed to bring the field to bit 0.
template <int BITS>
struct Scale {
    f16x2 step, z0, z1, z2;   // Step; 2^(10 - b) + Z for the field positions in use (b = 0, 4 / b = 0, 3, 6)
    float step_f;
    int z;
    bool packed;              // |Z| small enough for the packed path
    __device__ __forceinline__ void set(float s, int zero)
    {
        const _Float16 sh = (_Float16)s;
        step_f = (float)sh;
        z = zero;
        packed = zero >= -1024 && zero <= 1024;
        const _Float16 zh = (_Float16)(float)zero;
        const f16x2 zz = {zh, zh};
        step = f16x2{sh, sh};
        z0 = as_h2(0x64006400u) + zz;                                       // 1024 + Z
        z1 = as_h2(BITS == 4 ? 0x54005400u : 0x58005800u) + zz;             // 64 + Z / 128 + Z
        z2 = BITS == 4 ? z1 : as_h2(0x4c004c00u) + zz;                      // 16 + Z
    }
};

// The 24 bits of codes k = 8 d .. 8 d + 7 of the 32 (bits above them are not cleared)
__device__ __forceinline__ uint32_t fields3(const RawCodes<3>& rc, int d)
{
    return d == 0 ? rc.w[0] : d == 1 ? __builtin_amdgcn_alignbit(rc.w[1], rc.w[0], 24)
         : d == 2 ? __builtin_amdgcn_alignbit(rc.w[2], rc.w[1], 16) : rc.w[2] >> 8;
}

template <int BITS>
__device__ __forceinline__ uint32_t fields_of(const RawCodes<BITS>& rc, int d)   // codes k = 8 d .. 8 d + 7 of the 32
{
    if constexpr (BITS == 4) return rc.w[d];
    else return fields3(rc, d);
}

// (w & mask) | magic in one operation: the compiler spends two on literals, so they sit in registers it cannot see into
__device__ __forceinline__ uint32_t field(uint32_t w, uint32_t mask, uint32_t magic)
{
    asm("" : "+v"(mask));
    asm("" : "+s"(magic));
    return (w & mask) | magic;
}

// Eight codes (32 bits of INT4 / the low 24 bits of INT3) as four binary16 pairs (k, k + 4): (0,4) (1,5) (2,6) (3,7),
// the order the fields come out of the packed formats in (a caller that needs natural order permutes).
// 13 (INT4) / 16 (INT3) operations per 8 codes.
template <int BITS>
__device__ __forceinline__ void dequant_word(uint32_t w, const Scale<BITS>& s, uint32_t o[4])
{
    if constexpr (BITS == 4) {
        const uint32_t v = w >> 8;
        o[0] = as_u32((as_h2(field(w, 0x000f000fu, 0x64006400u)) - s.z0) * s.step);
        o[1] = as_u32((as_h2(field(w, 0x00f000f0u, 0x54005400u)) - s.z1) * s.step);
        o[2] = as_u32((as_h2(field(v, 0x000f000fu, 0x64006400u)) - s.z0) * s.step);
        o[3] = as_u32((as_h2(field(v, 0x00f000f0u, 0x54005400u)) - s.z1) * s.step);
    } else {
        // codes 4 .. 7 (bits 12 .. 23) move up by 4, so that both halves hold four fields at bits 0, 3, 6, 9
        const uint32_t g = (w & 0x0fffu) | ((w << 4) & 0x0fff0000u), h = g >> 9;
        o[0] = as_u32((as_h2(field(g, 0x00070007u, 0x64006400u)) - s.z0) * s.step);
        o[1] = as_u32((as_h2(field(g, 0x00380038u, 0x58005800u)) - s.z1) * s.step);
        o[2] = as_u32((as_h2(field(g, 0x01c001c0u, 0x4c004c00u)) - s.z2) * s.step);
        o[3] = as_u32((as_h2(field(h, 0x00070007u, 0x64006400u)) - s.z0) * s.step);
    }
}
// The same in natural order, (k, k + 1) (k + 2, k + 3) ...: INT4 brings each byte to both halves of a register, whose two
// fields then sit at bits 0 and 4; INT3 the codes of a pair to the same bit of the two halves (16 / 17 operations per 8 codes; INT3 by way of
// the other order 20: us, 256 tokens 4096 x 4096 23.6 -> 22.3, 11008 x 4096 44.5 -> 42.4, 17 tokens 4096 x 11008 13.9 -> 13.75)
__device__ __forceinline__ v4i natural_order(const uint32_t o[4]);
template <int BITS>
__device__ __forceinline__ v4i dequant_word_natural(uint32_t w, const Scale<BITS>& s)
{
    if constexpr (BITS == 4) {
        const f16x2 z01 = {s.z0.x, s.z1.x};
        v4i o;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const uint32_t b = __builtin_amdgcn_perm(w, w, 0x00010001u * (uint32_t)i);
            o[i] = (int)as_u32((as_h2(field(b, 0x00f0000fu, 0x54006400u)) - z01) * s.step);
        }
        return o;
    } else {
        // low half: codes from bit 0 (4: bit 12) on, high half: the same three bits further, so that both codes of a pair sit at bit 0 or 6
        const uint32_t a = __builtin_amdgcn_perm(w << 13, w, 0x07060100u), b = __builtin_amdgcn_perm(w << 1, w >> 12, 0x07060100u);
        return v4i{(int)as_u32((as_h2(field(a, 0x00070007u, 0x64006400u)) - s.z0) * s.step),
                   (int)as_u32((as_h2(field(a, 0x01c001c0u, 0x4c004c00u)) - s.z2) * s.step),
                   (int)as_u32((as_h2(field(b, 0x00070007u, 0x64006400u)) - s.z0) * s.step),
                   (int)as_u32((as_h2(field(b, 0x01c001c0u, 0x4c004c00u)) - s.z2) * s.step)};
    }
}
template <int BITS>
__device__ __forceinline__ void dequant8_pairs(const RawCodes<BITS>& rc, int d, const Scale<BITS>& s, uint32_t o[4])
{
    dequant_word<BITS>(fields_of<BITS>(rc, d), s, o);
}

// the same pairs for any zero point, through binary32
template <int BITS>
__device__ __forceinline__ void dequant_word_any(uint32_t w, const Scale<BITS>& s, uint32_t o[4])
{
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        int c[2];
#pragma unroll
        for (int e = 0; e < 2; ++e) c[e] = (int)((w >> (BITS * (q + 4 * e))) & ((1u << BITS) - 1u));
        const f16x2 h = {(_Float16)((float)(c[0] - s.z) * s.step_f), (_Float16)((float)(c[1] - s.z) * s.step_f)};
        o[q] = as_u32(h);
    }
}
template <int BITS>
__device__ __forceinline__ void dequant8_pairs_any(const RawCodes<BITS>& rc, int d, const Scale<BITS>& s, uint32_t o[4])
{
    dequant_word_any<BITS>(fields_of<BITS>(rc, d), s, o);
}

// pairs (k, k + 4) -> natural order (and back: the permutation of a 16-byte chunk of 8 halves is its own kind)
__device__ __forceinline__ v4i natural_order(const uint32_t o[4])
{
    return v4i{(int)__builtin_amdgcn_perm(o[1], o[0], 0x05040100u),    // k0 k1
               (int)__builtin_amdgcn_perm(o[3], o[2], 0x05040100u),    // k2 k3
               (int)__builtin_amdgcn_perm(o[1], o[0], 0x07060302u),    // k4 k5
               (int)__builtin_amdgcn_perm(o[3], o[2], 0x07060302u)};   // k6 k7
}
__device__ __forceinline__ v4i pair_order(v4i x)   // (k0 k1) (k2 k3) (k4 k5) (k6 k7) -> (0,4) (1,5) (2,6) (3,7)
{
    return v4i{(int)__builtin_amdgcn_perm((uint32_t)x[2], (uint32_t)x[0], 0x05040100u),
               (int)__builtin_amdgcn_perm((uint32_t)x[2], (uint32_t)x[0], 0x07060302u),
               (int)__builtin_amdgcn_perm((uint32_t)x[3], (uint32_t)x[1], 0x05040100u),
               (int)__builtin_amdgcn_perm((uint32_t)x[3], (uint32_t)x[1], 0x07060302u)};
}

}  // namespace wonly
}  // namespace aweq
