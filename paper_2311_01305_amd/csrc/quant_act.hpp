// The activation quantizer's launch and argument checks (quant_act.hip), for the entry points that run it first.
#pragma once
#include "equalize.hpp"

namespace aweq {

// colsum_xq in the form that the pass over the weights multiplies with: digits of four columns (code_digits.hpp) to an entry, and sums over
// kRangeCols channels each.  Fewer than 2^23 tokens.
struct SumDigits {
    uint4* digits;       // [K / 4]
    long long* totals;   // [ceil(K / kRangeCols)]
};

// range: Step and Z are not known yet, the launch derives and stores them (the panel form; asked for with colsum_xq only), on a workspace of
// quant_act_ws_bytes(T, K, true)
int launch_quant_act(const void* X, aweq_dtype dt, int64_t T, int64_t K, int64_t ldx, const float* inv_s,
                     const float* act_step, const int32_t* act_zero, int8_t* xq, int32_t* rowsum_x,
                     int64_t* colsum_xq, void* ws, uint32_t* status, hipStream_t st, const RangeParts* range = nullptr,
                     const SumDigits* digits = nullptr);
size_t quant_act_ws_bytes(int64_t T, int64_t K, bool fine = false);
int check_quant_act_ws(int64_t T, int64_t K, const int32_t* rowsum_x, const int64_t* colsum_xq, const void* ws, size_t ws_bytes);
int check_quant_act_args(const void* X, aweq_dtype dt, int64_t T, int64_t K, int64_t ldx, const float* inv_s,
                         const float* act_step, const int32_t* act_zero, const int8_t* xq, bool xq_optional);

}  // namespace aweq
