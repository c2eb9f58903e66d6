// Few-token form of the weight-only forward (gemm_wonly_small.hip), chosen by aweq_wonly_gemm.
#pragma once
#include "common.hpp"

namespace aweq {
namespace wonly {

struct SmallArgs {
    const _Float16* X;      // x_hat [T x K], row-major, pitch ldx
    const uint8_t* codes;
    const float* step;
    const int32_t* zero;
    const float* bias;
    void* out;
    int64_t ldx, ldo, T, N, K;
    uint32_t scale_pitch;   // (Step, Z) pairs per output channel: K / group, 1 (per row), 0 (per tensor)
    uint32_t group_magic;   // ceil(2^31 / (group / 32)): __umulhi(k / 16, it) = k / group for k a multiple of 32; 0 without groups
};

constexpr int64_t kSmallTokens = 256;

int launch_small(const SmallArgs& g, int bits, int group, bool out_f16, hipStream_t st);

}  // namespace wonly
}  // namespace aweq
