// The launcher of the matrix-core kernel (span_matrix.hip), called by the entry points in span_kernels.hip.
#ifndef SPAN_MATRIX_H_
#define SPAN_MATRIX_H_

#include "span_device.h"

namespace spanattn {

// Runs the call's base.q_len query tokens, p.tokens a launch, on `stream`; `base` holds the call's pointers and sizes.
hipError_t launch_matrix(const LaunchArgs& base, int dtype, int head_dim, const MatrixPlan& p, const uint32_t* table,
                         int batch, hipStream_t stream);

}  // namespace spanattn
#endif
