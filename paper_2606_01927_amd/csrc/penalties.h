// penalties.h -- internal interface between the C ABI (albireo.hip) and the standalone penalty kernel
// (penalties.hip).  Not part of the public header.
#pragma once

#include <stdint.h>

#include <hip/hip_runtime_api.h>

#include "albireo.h"

namespace albireo_penalties {

// Enqueue the penalties of B rows (params may be NULL) into out [B, V] fp32.  The caller has validated
// every host-checkable argument.
albireo_status_t launch(const void* logits, albireo_dtype_t dtype, int64_t B, int64_t V, int64_t ld,
                        const albireo_params_t* params, float* out, hipStream_t stream);

}  // namespace albireo_penalties
