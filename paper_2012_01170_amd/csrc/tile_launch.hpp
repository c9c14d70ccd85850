// The launch of the contraction's kernel for one basis size and tile height.
#pragma once

#include "tile_args.hpp"
#include "tile_kernels.hpp"

namespace sbc {

// Registers: given values of 24 and 32 functions spill (65 to 157, and 320 to 353:
// the sums of all functions of 16 rows are held at once), bf16 of M = 8 and 10 with
// tall tiles 8 to 13.  Shapes that lose by it go to the separate kernels
// (route_cost.hpp).
template <int M, bool kXbf, StageKind kKind, bool kTall>
void launch_contract(const TileContractArgs &a, hipStream_t s) {
    const int32_t tiles = grid_for(a.p.n_rows, kTall && kAlwaysTall<kKind> ? 64 : 32);
    const int32_t cols = contract_columns(tiles, a.N);
#define SBC_TILE(NCBW, WCB)                                                                      \
    hipLaunchKernelGGL((tile_contract_kernel<M, kXbf, kKind, kTall, NCBW, WCB>),                 \
                       dim3((unsigned)tiles, (unsigned)((a.N + cols - 1) / cols)),               \
                       dim3(kTileThreads), 0, s, a.p, a.v, a.g, a.mode, a.X, a.C, a.frag, a.N,   \
                       a.out)
    // (column blocks of 16 over the waves)
    if (cols == 32) SBC_TILE(2, 1);
    else if (cols == 64) SBC_TILE(2, 2);
    else if constexpr (M < 10 || !kTall) SBC_TILE(4, 2);
#undef SBC_TILE
}

}  // namespace sbc
