// Internal launchers of the two prefill kernels (Eq. 2).
#pragma once

#include <hip/hip_runtime.h>

#include "tca_common.h"
#include "tca_device.h"

namespace tca {

// fp32 storage: fp64 logits, fp32 exponentials and accumulation.
int launch_prefill_f32(const tca_params* prm, const float* Q, int64_t q_pos0, int64_t n_queries, const float* K,
                       const float* V, int64_t kv_stride, const int32_t* idx, const float* Kg, const float* Vg,
                       const int64_t* offs, const int32_t* n_rows, float* O, float* lse, hipStream_t st, int part);

// bf16 MFMA flash kernel.
// _bytes: the workspace a caller is told to bring; _need: what a call must have.  The rest holds the partial results
// of calls cut into chunks of keys, which a smaller workspace has fewer or none of.
size_t prefill_mfma_workspace_bytes(const tca_params* prm, int64_t n_queries, int64_t cap_rows);
size_t prefill_mfma_workspace_need(const tca_params* prm, int64_t n_queries, int64_t cap_rows);
int launch_prefill_mfma(const tca_params* prm, const bf16_t* Q, int64_t q_pos0, int64_t n_queries,
                        const bf16_t* K, const bf16_t* V, int64_t kv_stride, const int32_t* idx,
                        const bf16_t* Kg, const bf16_t* Vg, const int64_t* offs, const int32_t* n_rows,
                        bf16_t* O, float* lse, void* ws, size_t ws_bytes, hipStream_t st, int part);
// Calls with too few query tiles for the chip: the tiles of a (head, query tile) item are cut into chunks of
// `chunk` tiles, one workgroup each, whose unnormalised results launch_merge_split combines.
struct SplitPlan {
  float* part;                          // per workgroup: the O^T accumulators, then m and l of its queries
  int32_t chunk;                        // tiles per chunk, even
  int32_t run;                          // consecutive workgroups that go to one XCD
  int32_t item_start[TCA_MAX_HEADS + 1];  // head h's workgroups: [item_start[h], item_start[h + 1]), chunk-major, query tiles inside
};
template <int D> constexpr size_t split_floats() { return 128 * (size_t)(D + 2); }      // per workgroup of 128 queries
// O = bf16 [Hq, n_queries, D], lse as for tca_prefill (may be NULL).
void launch_merge_split(const tca_params* prm, const SplitPlan& sp, int64_t n_queries, uint16_t* O, float* lse, hipStream_t st);
// The ranges of the (head, query tile) sequence the eight XCDs work through for such a call
// (start_out[9]); returns the number of workgroups launched, -1 if the head count is not a multiple of 8.
int64_t prefill_mfma_xcd_plan(const tca_params* prm, const int64_t* offs, int64_t q_pos0, int64_t n_queries, int part,
                              bool gather, int32_t* start_out);
// What tca_diag_prefill_walk returns.
int prefill_mfma_walk(const tca_params* prm, const int64_t* offs, int64_t q_pos0, int64_t n_queries, int part, bool gather,
                      size_t ws_bytes, int32_t* heads_out, int64_t* chunks_out);

}  // namespace tca
