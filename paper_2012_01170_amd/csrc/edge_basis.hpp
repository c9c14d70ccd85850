// Basis values of one edge inside the kernels that gather along the pattern,
// and the geometry they read.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

#include "../../include/sbconv.h"
#include "basis.hpp"

namespace sbc {

// ---------------------------------------------------------------- geometry
// Geometry as the fused kernels read it: the caller's point coordinates, and
// for event streams a packed copy (px, py, t, 0) per event, so that one
// 16-byte load brings all three coordinates of an edge's far end (three
// separate arrays would cost three cache lines per edge).
struct KGeo {
    double inv_r;
    float inv_tau;
    int32_t nnz;  // edge bound of the pattern: row extents are clamped to [0, nnz]
    const float *x_in, *x_out;
    const int4 *ev;
    const float *decays;  // learned-decay rates [8, M / 8]
    const double *wsum;   // weighted basis: the weight sum W_i of every output row
};

// Basis mode of the fused kernels for the derivatives of the learned-decay
// basis with respect to its rates (the decay gradient's D-route pass).
constexpr int kDecayDerivMode = 16;

// Basis mode of the backward for the fixed-decay event basis when the
// gathered rows, the packed events or the pattern arrays pass 4 GiB: the
// generic gather (64-bit addressing) instead of the one-hot gather, whose
// loads take 32-bit byte offsets from their arrays' bases.
constexpr int kEvent8WideMode = 17;
// The same for the learned-decay basis and its derivatives (M / 8 values per
// edge), whose in-place gather takes 32-bit byte offsets too.
constexpr int kDecaysWideMode = 18;
constexpr int kDecayDerivWideMode = 19;

// ---------------------------------------------------------------- basis per edge
// kBasis: 0 = read v[ev, :], SBC_BASIS_MONO4 + 1, SBC_BASIS_MONO8 + 1, SBC_BASIS_EVENT8 + 1,
// SBC_BASIS_EVENT_DECAYS + 1 (M / 8 rates per offset), kDecayDerivMode (their
// derivatives with respect to the rates) (i = output index, j = input index
// of the edge, ev = its CSR position).
template <int M, int kBasis>
__device__ __forceinline__ void edge_basis(const KGeo &g, const float *__restrict__ v,
                                           int32_t i, int32_t j, int64_t ev, double inv_r,
                                           float inv_tau, float *out) {
    if constexpr (kBasis == 0) {
#pragma unroll
        for (int m = 0; m < M; ++m) out[m] = v[ev * M + m];
    } else if constexpr (kBasis == SBC_BASIS_EVENT8 + 1 || kBasis == kEvent8WideMode) {
        const int4 a = g.ev[i], b = g.ev[j];
        const int k = event_index(a.x - b.x, a.y - b.y);
        const float d = event_decay(a.z, b.z, inv_tau);
#pragma unroll
        for (int m = 0; m < M; ++m) out[m] = (m == k) ? d : 0.f;
    } else if constexpr (kBasis == SBC_BASIS_EVENT_DECAYS + 1 || kBasis == kDecayDerivMode) {
        // the same expression as the basis values kernel, so the values agree bitwise
        constexpr int Mv = M / 8;
        const int4 a = g.ev[i], b = g.ev[j];
        const int k = event_index(a.x - b.x, a.y - b.y);
        const float dt = (float)((int64_t)a.z - (int64_t)b.z);
        float x[Mv];
#pragma unroll
        for (int q = 0; q < Mv; ++q) {
            x[q] = k >= 0 ? expf(-g.decays[k * Mv + q] * dt) : 0.f;
            if (kBasis == kDecayDerivMode) x[q] = -dt * x[q];
        }
#pragma unroll
        for (int m = 0; m < M; ++m) out[m] = (m / Mv == k) ? x[m % Mv] : 0.f;
    } else {
        point_basis<M>(g.x_out[3 * (int64_t)i], g.x_out[3 * (int64_t)i + 1],
                       g.x_out[3 * (int64_t)i + 2], g.x_in[3 * (int64_t)j],
                       g.x_in[3 * (int64_t)j + 1], g.x_in[3 * (int64_t)j + 2], inv_r, out);
    }
}

}  // namespace sbc
