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
// The ranges of the (head, query tile) sequence the eight XCDs work through for such a call
// (start_out[9]); returns the number of workgroups launched, -1 if the head count is not a multiple of 8.
int64_t prefill_mfma_xcd_plan(const tca_params* prm, const int64_t* offs, int64_t q_pos0, int64_t n_queries, int part,
                              bool gather, int32_t* start_out);

}  // namespace tca
