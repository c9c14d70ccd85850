// The launch of the contraction's kernel for one basis size and tile height.
#pragma once

#include "tile_args.hpp"
#include "tile_kernels.hpp"

namespace sbc {

// Columns a block takes: N rounded up to 32, 64 or 128, halved while twice the
// blocks still leave a CU to each.  The blocks of a row tile gather for
// themselves, but on CUs that would idle, and each multiplies fewer columns
// (256 rows, M 8, 64 -> 128 channels, 5 entries a row: 25.6 -> 18.4 us).  With two
// blocks a CU the gathers got in each other's way (4096 rows, 45 entries: 59 us
// in blocks of 128 columns, 57 of 64, 66 of 32).
inline int32_t contract_columns(int32_t tiles, int32_t N) {
    int32_t w = N <= 32 ? 32 : N <= 64 ? 64 : 128;
    while (w > 32 && (int64_t)tiles * ((N + w / 2 - 1) / (w / 2)) <= 256) w /= 2;
    return w;
}

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
