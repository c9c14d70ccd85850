// Arguments and launches of the tile passes' kernels, by basis size (the
// instantiations are compiled apart, one source per group of sizes).
#pragma once

#include "tile.hpp"

namespace sbc {

struct TileContractArgs {
    TilePattern p;
    const float *v;
    KGeo g;
    int mode;
    const void *X;
    int32_t C;
    const uint16_t *frag;
    int32_t N;
    float *out;
    bool tall;  // tiles of 64 rows where the rows are short (M <= 10 only)
};

struct TileDwArgs {
    TilePattern p;
    const float *v;
    KGeo g;
    int mode;
    const void *P;
    int32_t CP;
    const void *Q;
    int32_t CQ;
    float *part;
    int32_t splits;
};

// Channels per slice, and blocks of 16 channels of a P chunk
constexpr int32_t kTileCS = 32;
constexpr int32_t dw_npb(int32_t M, int32_t CP) { return M >= 16 || CP <= 32 ? 2 : 4; }

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

// Parts that the rows of a weight gradient are split into: two blocks per CU with
// the chunks and slices of its channels.
inline int32_t dw_splits(int32_t n_rows, int32_t M, int32_t CP, int32_t CQ) {
    const int32_t pc = 16 * dw_npb(M, CP);
    const int64_t ny = (int64_t)((CQ + kTileCS - 1) / kTileCS) * ((CP + pc - 1) / pc);
    const int64_t tiles = ((int64_t)n_rows + 31) / 32;
    int64_t s = 512 / ny;
    if (s > tiles) s = tiles;
    return s < 1 ? 1 : (int32_t)s;
}

sbc_status launch_contract_4_8_10(int32_t M, bool bf16, const TileContractArgs &a, hipStream_t s);
sbc_status launch_contract_16_24_32(int32_t M, bool bf16, const TileContractArgs &a, hipStream_t s);
sbc_status launch_dw(int32_t M, bool bf16, const TileDwArgs &a, hipStream_t s);

}  // namespace sbc
