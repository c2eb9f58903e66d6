// One pass over the weights of a calibration: fold (Eq. 3), quantise (Eq. 1-2) and correct the bias (Eq. 11-15) from registers
// (weight_pass.hip).
#pragma once
#include "equalize.hpp"

namespace aweq {

constexpr int kMaxMembers = 4;   // weights that share one input

struct PassMember {
    const void* W;
    void* W_hat;
    uint8_t* codes;
    float* step;
    int32_t* zero;
    int32_t* rowsum;        // 8 bits; nullable
    const float* bias_in;   // nullable
    float* delta;
    float* bias_out;
    long long* colsum_acc;  // 8 bits; nullable
    int64_t N, ldw, ldwh;
    unsigned first_block;   // set by the launch
};

// What a calibration derives from the pieces of the ranges besides Step and Z: R and p = r / R (Eq. 4) of activations and weights
struct FinishArgs {
    RangeParts range;   // act_step null: xhat_range, Step and Z are written elsewhere
    const float *r_x, *r_w;
    float *R_x, *R_w, *p_x, *p_w;   // p nullable
    const int32_t* colsum;          // nullable: its copies' sum is widened to colsum_xq
    long long* colsum_xq;
    uint32_t* status;
};

struct PassArgs {
    PassMember m[kMaxMembers];
    int n;
    unsigned weight_blocks;   // the blocks behind them do `fin`; set by the launch
    int64_t K;
    const float* s;
    const float* mu;
    uint64_t count;                // 8 bits: tokens behind colsum_xq
    const int32_t* colsum;         // 8 bits: colsum_xq, of fewer than 2^23 tokens, as the sum of `copies` rows (beyond kCopiesK columns one)
    int copies;
    const float* act_step;         // 8 bits
    const int32_t* act_zero;
    int enable_bc;
    uint32_t* status;
    FinishArgs fin;
};

// shapes the pass takes: 8 bits per row (the int8 path), 4 / 3 bits per group (weight-only)
bool weight_pass_takes(int bits, int group, bool w8a8, int64_t N, int64_t K, uint64_t count);
int launch_weight_pass(PassArgs& a, aweq_dtype dt, int bits, int group, hipStream_t st);
// `fin` alone
int launch_finish(const FinishArgs& fin, int64_t K, hipStream_t st);

}  // namespace aweq
