// Forms of the weight-only forward for fewer tokens (gemm_wonly_small.hip, gemm_wonly_mid.hip) that aweq_wonly_gemm chooses from.
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

// The few-token kernel's channels per workgroup (16 times nt) for a shape, and what it is modelled to take: us at K = 8192 (every
// kernel's time is close to proportional to K)
struct SmallPlan {
    int nt;
    double cost;
};
SmallPlan plan_small(int64_t T, int64_t N);
int launch_small(const SmallArgs& g, int bits, int group, const SmallPlan& p, bool out_f16, hipStream_t st);

// The same of the kernel for some hundred tokens (gemm_wonly_mid.hip), which takes groups that are multiples of 128, one (Step, Z)
// per row or one per tensor, and pitches whose 128 rows lie within 2^32 bytes (32-bit byte offsets inside a tile of rows)
struct MidPlan {
    bool square;   // 128 x 128 tiles instead of 64 x 128
    double cost;
};
MidPlan plan_mid(int64_t T, int64_t N);
int launch_mid(const SmallArgs& g, int bits, const MidPlan& p, bool out_f16, hipStream_t st);

}  // namespace wonly
}  // namespace aweq
