// What the evaluation orders of a convolution take, in microseconds on an
// MI355X, from its sizes alone: the choice between the tile passes (tile.hpp)
// and the separate gathers and contractions (spmm.hpp, gemm.hpp).
//
// The tile pass gathers a row tile again for every chunk of result columns (the
// weight gradient: of P channels) and pays for it per entry and basis function;
// the separate kernels gather once and move M C floats a row through memory
// instead.  So neither serves all sizes: 32768 rows, M 8, 5.7 entries a row, 512
// -> 128 channels 236 us against 405, and 512 -> 8 with 20 entries 322 against
// 128 contracting first; 24 values a row given, 20 entries, 64 -> 64, both
// gradients 704 against 338.
//
// The coefficients are least-squares fits (of the relative error) to 4632
// measured shapes: 64 to 32768 rows, 4 to 45 entries a row, 8 to 512 channels,
// every M, bases and values, both types; half of the times are met within 12 %,
// nine tenths within 30 %.  Over them the choice is 1.9 % from the best of the
// routes in the mean, and slower by 5 % or more than the better of the separate
// ones in 7 % of the shapes, where the tile passes alone were in 55 %.
#pragma once

#include <cstdint>

#include "tile_args.hpp"

namespace sbc {

// A convolution: R rows that gather E entries of C channels, N result channels.
struct RouteSize {
    int32_t R;
    int64_t E;
    int32_t M, C, N;
};

// One contraction: a block of rows walks its channels in slices of 32; blocks
// beyond the 512 that the CUs hold at once wait their turn.  values: the basis
// values are given (rows of 24 and 32 of them cost more than evaluated ones).
inline double tile_contract_us(const RouteSize &s, bool bf16, bool values) {
    const int32_t M = s.M, tiles = (int32_t)(((int64_t)s.R + 31) / 32);
    const int32_t w = contract_columns(tiles, s.N);
    const double turns = 1.0 + (double)tiles * ((s.N + w - 1) / w) / 512.0;
    const double deg = s.R > 0 ? (double)s.E / s.R : 0.0;
    const double row = M <= 10 ? 0.024 + 0.0023 * M : M == 16 ? 0.07 : M == 24 ? 0.1 : 0.155;
    const double entry = M <= 10   ? 0.0021 + 0.00032 * M
                         : M == 16 ? 0.0107
                         : M == 24 ? (values ? 0.0204 : 0.0147)
                                   : (values ? 0.0423 : 0.0175);
    const double product = M * w * (bf16 ? 7e-5 : 1.1e-4);
    const int32_t Cp = (s.C + kTileCS - 1) / kTileCS * kTileCS;
    return 10.0 + turns * Cp * (row + entry * deg + product);
}

// One weight gradient over R rows of C_P channels that gather C_Q (C, N: those).
inline double tile_dw_us(const RouteSize &s, bool bf16, bool values) {
    const int32_t M = s.M, CP = s.C, CQ = s.N, npb = dw_npb(M, CP);
    const double ny = (double)((CP + 16 * npb - 1) / (16 * npb)) * ((CQ + kTileCS - 1) / kTileCS);
    const double tiles = (double)(((int64_t)s.R + 31) / 32), splits = dw_splits(s.R, M, CP, CQ);
    const double deg = s.R > 0 ? (double)s.E / s.R : 0.0;
    const double tile = M <= 10 ? 0.55 + (0.05 + 0.0155 * M) * deg +
                                      M * (0.04 + (bf16 ? 0.035 : 0.06) * npb)
                        : M == 16 ? (values ? 0.38 : 0.3) * deg + 2.4
                        : M == 24 ? (values ? 1.16 : 0.67) * deg + 6.0
                                  : (values ? 1.9 : 0.85) * deg + 8.5;
    return 12.0 + tiles / splits * (1.0 + splits * ny / 512.0) * tile +
           splits * CP * M * CQ * (M == 32 ? 3e-6 : 1.2e-6);
}

// The separate kernels: sums over entries, rows and products, and the serial
// gather of one row's entries, which few rows leave exposed (`deg` of them).
inline double mean_degree(int64_t nnz, int32_t rows) { return rows > 0 ? (double)nnz / rows : 0.0; }

// (N F) W: R rows gather C channels, then contract.
inline double split_forward_us(const RouteSize &s) {
    const double E = (double)s.E, M = s.M, MC = M * s.C, MCN = MC * s.N;
    return 18.0 +
           1e-5 * (0.57 * E * M + 0.015 * E * s.C + 0.0067 * E * MC + 0.16 * s.R * MC +
                   0.0018 * s.R * MCN + 0.42 * MCN + 60.0 * MC) +
           mean_degree(s.E, s.R) * (5.7e-4 * s.C + 7.5e-5 * MC);
}

// N (F W): R_in rows contract, then the entries gather N channels.
inline double gemm_first_forward_us(const RouteSize &s, int32_t R_in) {
    const double E = (double)s.E, M = s.M, MN = M * s.N, MCN = MN * s.C;
    return 18.0 +
           1e-5 * (0.55 * E * M + 0.019 * E * MN + 0.2 * R_in * MN + 0.0017 * R_in * MCN +
                   0.79 * MCN + 850.0 * s.C) +
           mean_degree(s.E, s.R) * (9.5e-4 * s.N + 1.3e-4 * MN);
}

// Both gradients of C_in -> C_out: the D-route (n_in rows gather C_out
// channels) and the G-route (n_out rows gather C_in).
inline double split_d_us(int32_t n_in, int64_t nnz, int32_t M_, int32_t Ci, int32_t Co) {
    const double E = (double)nnz, M = M_, MN = M * Co, MCN = MN * Ci;
    return 31.0 +
           1e-5 * (0.71 * E * M + 0.027 * E * Co + 0.006 * E * MN + 0.23 * n_in * MN +
                   0.0037 * n_in * MCN + 1.4 * MCN + 140.0 * MN + 28.0 * n_in) +
           mean_degree(nnz, n_in) * (7.2e-4 * Co + 1.05e-4 * MN);
}
inline double split_g_us(int32_t n_out, int64_t nnz, int32_t M_, int32_t Ci, int32_t Co) {
    const double E = (double)nnz, M = M_, MC = M * Ci, MCN = MC * Co;
    return 27.0 +
           1e-5 * (1.1 * E * M + 0.03 * E * MC + 0.38 * n_out * MC + 0.0039 * n_out * MCN +
                   0.96 * MCN + 910.0 * Co + 40.0 * n_out) +
           mean_degree(nnz, n_out) * (2.1e-3 * Ci + 2.7e-4 * MC);
}

// The weight gradient alone over n_out rows that gather C_in channels.
inline double split_dw_us(int32_t n_out, int64_t nnz, int32_t M_, int32_t Ci, int32_t Co) {
    const double E = (double)nnz, M = M_, MC = M * Ci, MCN = MC * Co;
    return 19.0 +
           1e-5 * (0.53 * E * M + 0.015 * E * Ci + 0.0076 * E * MC + 0.16 * n_out * MC +
                   0.002 * n_out * MCN + 0.19 * MCN + 29.0 * n_out) +
           mean_degree(nnz, n_out) * (4e-4 * Ci + 7e-5 * MC);
}

// The separate kernels are taken where they are estimated this much faster: at
// equal times the tile pass needs no intermediate in memory and its split
// products lose less.  Of 593 measured layers of up to 128 channels and 25 entries
// a row with evaluated bases, forward and gradients together, 0.9 leaves 26 more
// than 3 % slower than the tile passes and 41 than the separate kernels (0.95: 66
// and 41, 0.85: 10 and 60).
constexpr double kTileFavour = 0.9;

}  // namespace sbc
