// Fused forward / backward kernels (fused.hip).
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

#include "../../include/sbconv.h"
#include "edge_basis.hpp"

namespace sbc {

// Upper bound on the persistent blocks of the fused backward (one per CU).
constexpr int kMaxBlocksBwd = 256;

bool fused_forward_available(int32_t M, int32_t CI, int32_t CO, bool bf);
bool fused_backward_available(int32_t M, int32_t CI, int32_t CO, bool bf);
// n_points: the larger of the input and output counts
size_t fused_workspace_bytes(int32_t M, int32_t CI, int32_t CO, int32_t n_points);
// the forward's
size_t fused_forward_workspace_bytes(int32_t n_points);

// Kernel geometry of a call; `packed` (16 bytes per event) receives the packed
// coordinates of an event stream whose basis is evaluated inside the kernels.
sbc_status make_kgeo(const sbc_csr *csr, const float *v, const sbc_geometry *g, void *packed,
                     hipStream_t stream, KGeo *kg);

// Y = sum_m N^(m) F W^(m) in one kernel (plus the order of its rows).
sbc_status fused_forward(const sbc_csr *csr, const float *v, const sbc_geometry *g, int32_t M,
                         const void *F, const void *W, bool bf, int32_t CI, int32_t CO, float *Y,
                         void *ws, hipStream_t stream);

// dF and/or dW (either may be null) by the transposed gather D = N^T dY.
sbc_status fused_backward(const sbc_csr *csr, const sbc_csc *csc, const float *v,
                          const sbc_geometry *g, int32_t M, const void *F, const void *W,
                          const void *dY, bool bf, int32_t CI, int32_t CO, float *dF, float *dW,
                          void *ws, hipStream_t stream, bool decay_derivative = false);

}  // namespace sbc
