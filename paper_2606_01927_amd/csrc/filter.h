// filter.h -- internal interface between the C ABI (albireo.hip) and the filtered-distribution kernels
// (filter.hip).  Not part of the public header.
#pragma once

#include <stddef.h>
#include <stdint.h>

#include <hip/hip_runtime_api.h>

#include "albireo.h"

namespace albireo_filter {

// Workspace bytes of a call (at most what albireo_workspace_size reports for fp32 rows), 0 when the shape
// is not served here.
size_t workspace_bytes(int64_t B, int64_t V);

// Enqueue albireo_topk_topp on rows of V fp32 logits.  The caller has validated every host-checkable
// argument; ws holds workspace_bytes(B, V) zero bytes and is left zero.
albireo_status_t launch(const float* logits, int64_t B, int64_t V, int64_t ld, const albireo_params_t* params,
                        float* out_probs, float* out_threshold, int32_t* out_kept, float* out_log_norm,
                        uint32_t* out_flags, unsigned char* ws, hipStream_t stream);

}  // namespace albireo_filter
