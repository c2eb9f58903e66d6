// One pass over the weights of a calibration: fold (Eq. 3), quantise (Eq. 1-2) and correct the bias (Eq. 11-15) from registers
// (weight_pass.hip).
#pragma once
#include "equalize.hpp"

namespace aweq {

constexpr int kMaxMembers = 4;   // weights that share one input

// Copies of the activation codes' column sums that the quantizer's blocks add to in turn: many blocks to a column of a narrow matrix wait for each
// other (us, whole calibrations, one copy -> four: 65536 tokens 512 x 512 58.4 -> 45.4, 30000 tokens with the forward 74.3 -> 61.8, binary32 2048 tokens 25.5 ->
// 24.1, 262144 tokens 1024 x 1024 193 -> 187).  Beyond 1024 columns, where the pass over the weights has no registers for more, one: four copies of 4096
// columns 63.0 -> 64.1 with 9000 tokens; with one copy such calls wait too, but less than a merge takes (partial rows and a merge -> one copy: 1032 columns of
// 32768 / 131072 / 262144 tokens 56.8 -> 52.9 / 152 -> 147 / 270 -> 264, 2048 columns 71.1 -> 66.0 / 201 -> 197 / 362 -> 360).
constexpr int64_t kCopiesK = 1024;
constexpr int kMostCopies = 4;
inline int sum_copies(int64_t K) { return K <= kCopiesK ? kMostCopies : 1; }
// Up to so many tokens one copy: few blocks add to a column, and three copies less have to be zeroed, then read by every wavefront of the pass over the
// weights (us, whole calibrations of 512 channels, four -> one: 256 tokens K = 512 18.6 -> 17.7, K = 1024 20.6 -> 18.9, 1024 tokens 18.8 -> 18.6 and 22.0 -> 20.8,
// 1536 tokens 19.4 -> 19.5 and 23.1 -> 22.1, 2048 tokens 19.9 -> 20.6 and 23.2 -> 23.3, 4096 tokens 22.6 -> 25.4 and 25.3 -> 25.6; binary32 within 1 % of the same)
inline int64_t copies_tokens(int64_t K) { return K <= 512 ? 1280 : 2048; }

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
