// The activation quantizer's launch and argument checks (quant_act.hip), for the entry points that run it first.
#pragma once
#include "equalize.hpp"

namespace aweq {

// range: Step and Z are not known yet, the launch derives and stores them (the panel form).  colsum_added [copies][K], asked for with range and only then: the blocks add
// their sums over tokens to one of its rows and, where quant_act_adds_rows, a row's sums to rowsum_x, both zero before the launch, and nothing merges them; in the place
// of colsum_xq and ws.  Fewer than 2^23 tokens.
int launch_quant_act(const void* X, aweq_dtype dt, int64_t T, int64_t K, int64_t ldx, const float* inv_s,
                     const float* act_step, const int32_t* act_zero, int8_t* xq, int32_t* rowsum_x,
                     int64_t* colsum_xq, void* ws, uint32_t* status, hipStream_t st, const RangeParts* range = nullptr,
                     int32_t* colsum_added = nullptr, int copies = 1);
bool quant_act_adds_rows(int64_t K);   // with colsum_added: a row's sum comes from several blocks
size_t quant_act_ws_bytes(int64_t T, int64_t K);
int check_quant_act_ws(int64_t T, int64_t K, const int32_t* rowsum_x, const int64_t* colsum_xq, const void* ws, size_t ws_bytes);
int check_quant_act_args(const void* X, aweq_dtype dt, int64_t T, int64_t K, int64_t ldx, const float* inv_s,
                         const float* act_step, const int32_t* act_zero, const int8_t* xq, bool xq_optional);

}  // namespace aweq
