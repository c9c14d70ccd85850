// Tile passes of the convolution for any channel counts (tile*.hip).
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

#include "../../include/sbconv.h"
#include "edge_basis.hpp"

namespace sbc {

// A pattern as a tile pass walks it: rows r with entries ptr[r] .. ptr[r+1],
// the other end of entry e in idx[e] and its basis values' row perm[e] (or e).
// transposed: the rows are the convolution's inputs (a CSC).
struct TilePattern {
    int32_t n_rows;
    const int32_t *ptr, *idx, *perm;
    bool transposed;
};

// Whether the tile passes take a convolution of these sizes.
bool tile_available(int32_t M, int32_t C_in, int32_t C_out);

// out[r, n] = sum over m, c of (sum over row r's entries of value m times
// X[other, c]) B[m, c, n]: the forward (X = F, B = W), or the input gradient
// (transposed pattern, X = dY, B[m, c, n] = W[m, n, c]).  mode: basis mode
// (edge_basis.hpp); frag: tile_frag_bytes(M, C, N, bf16) of workspace.
size_t tile_frag_bytes(int32_t M, int32_t C, int32_t N, bool bf16);
sbc_status tile_contract(const TilePattern &p, const float *v, const KGeo &g, int mode, int32_t M,
                         const void *X, const void *W, bool w_transposed, bool bf16, int32_t C,
                         int32_t N, float *out, void *frag, hipStream_t stream, const char *trace);

// dW [M, C_in, C_out] = sum over rows r of P[r, :]^T (x) (the gathered sums of
// row r over Q).  Pattern transposed: P = F, Q = dY; else P = dY, Q = F.
// part: tile_dw_bytes() of workspace.
size_t tile_dw_bytes(int32_t n_rows, int32_t M, int32_t C_P, int32_t C_Q);
sbc_status tile_weight_gradient(const TilePattern &p, const float *v, const KGeo &g, int mode,
                                int32_t M, const void *P, const void *Q, bool bf16, int32_t C_in,
                                int32_t C_out, float *dW, void *part, hipStream_t stream,
                                const char *trace);

}  // namespace sbc
