// Arguments of the int8 GEMM kernels, and the forms for fewer tokens (gemm_i8_few.hip, gemm_i8_mid.hip) that
// aweq_w8a8_gemm chooses from.
#pragma once
#include "tile_walk.hpp"

namespace aweq {

struct GemmArgs : TileWalk {
    const int8_t* A;   // xq [T x K], K-panel layout
    const int8_t* B;   // wq [N x K], K-panel layout
    int64_t T, N, K;
    int32_t* out_i32;
    void* out_deq;
    int out_f16;
    int64_t ldo;
    long long* colsum_acc;
    const float* act_step;
    const int32_t* act_zero;
    const float* step_w;
    const int32_t* zero_w;
    const int32_t* rowsum_x;
    const int32_t* rowsum_w;
    const float* bias;
    int w_per_tensor;  // step_w / zero_w hold one entry for the whole weight instead of one per output channel
    // fused epilogues on the de-quantised binary16 output y (the next layer's calibration input)
    int act;                    // 0: none, 1: ReLU before y is rounded
    uint32_t* ykeys;            // [2 N] order-preserving keys of the column minimum / maximum of y
    long long* yfix;            // [N] column sums of y in units of 2^-24 (exact: y is binary16)
    const float* next_inv_s;    // [N] the next layer's 1 / s, Step and Z: y is quantised with them
    const float* next_step;
    const int32_t* next_zero;
    int8_t* yq;                 // [T x N] codes of y, K-panel layout (panels of 64 output channels)
    int32_t* rowsum_y;          // [T]
    long long* colsum_yq;       // [N]
    uint32_t* status;
};

// Several weights of N channels each that multiply the same codes, in one launch of the tiled kernel: the tile columns of one after the other's
// (TileWalk's), each weight with its own operands and output; B, out_deq, step_w, zero_w, rowsum_w and bias above are not read.
constexpr int kGroupMost = 4;
struct GroupArgs : GemmArgs {
    struct Member {
        const int8_t* B;
        void* out_deq;
        const float* step_w;
        const int32_t* zero_w;
        const int32_t* rowsum_w;
        const float* bias;
    } m[kGroupMost];
    int member_tiles;   // tile columns of a weight
};

// The binary16 outputs of n weights of N channels (g: what they share; K, T and A among it) in one launch, where it is modelled to take less than a
// launch each; AWEQ_ERR_SHAPE, and nothing launched, where not
int launch_gemm_i8_group(GroupArgs& g, int n, hipStream_t st);

// The few-token kernel's tile for a shape, and what it is modelled to take in the unit of kTiledRoundCost
struct FewPlan {
    int tile;      // index of the instantiation
    double cost;
};
FewPlan plan_few(int64_t T, int64_t N);
int launch_gemm_i8_few(const GemmArgs& g, const FewPlan& p, hipStream_t st);

// The same for at most kQuantTokens binary16 / binary32 tokens that the launch quantises itself (what the activation quantizer would
// write goes to xq and rowsum_x; g.A and g.rowsum_x are not read)
struct QuantIn {
    const void* X;
    int64_t ldx;
    const float* inv_s;
    int8_t* xq;
    int32_t* rowsum_x;
};
int launch_gemm_i8_few_quant(const GemmArgs& g, const FewPlan& p, const QuantIn& in, bool f16, hipStream_t st);
constexpr int kQuantTokens = 4;
constexpr int64_t kQuantFewBytes = 16384;   // codes such a launch may hold

// The same of the kernel for some hundred tokens (gemm_i8_mid.hip)
struct MidPlan {
    bool square;   // 128 x 128 tiles instead of 64 x 128
    double cost;
};
MidPlan plan_mid(int64_t T, int64_t N);
int launch_gemm_i8_mid(const GemmArgs& g, const MidPlan& p, hipStream_t st);

// Time of one round of workgroups at K = 8192 (us; every kernel's time is close to proportional to K): 256 tiles of 256 x 256
constexpr double kTiledRoundCost = 100.0;
constexpr double kHalfTileCost = 0.57;   // the same of 128 x 256 tiles, against that (0.55 - 0.58 from K = 256 to 16384)

}  // namespace aweq
