// The launch of the contraction's kernel for one basis size and tile height.
#pragma once

#include "tile_args.hpp"
#include "tile_kernels.hpp"

namespace sbc {

template <int M, bool kXbf, StageKind kKind, int TR>
void launch_contract(const TileContractArgs &a, hipStream_t s) {
    const int32_t ncb = (a.N + 15) / 16;
    const unsigned tiles = (unsigned)grid_for(a.p.n_rows, TR);
#define SBC_TILE(NCBW, WCB)                                                                      \
    hipLaunchKernelGGL((tile_contract_kernel<M, kXbf, kKind, TR, NCBW, WCB>),                            \
                       dim3(tiles, (unsigned)((ncb + NCBW * WCB - 1) / (NCBW * WCB))),            \
                       dim3(kTileThreads), 0, s, a.p, a.v, a.g, a.mode, a.X, a.C, a.frag, a.N,    \
                       a.out)
    // column blocks of 16 over the waves: the fewest that cover N, 128 at most
    if (ncb <= 2) SBC_TILE(2, 1);
    else if (ncb <= 4) SBC_TILE(2, 2);
    else if constexpr (M < 10 || TR == 32) SBC_TILE(4, 2);
#undef SBC_TILE
}

}  // namespace sbc
