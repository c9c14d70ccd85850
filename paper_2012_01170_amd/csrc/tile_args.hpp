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

sbc_status launch_contract_4_8_10(int32_t M, bool bf16, const TileContractArgs &a, hipStream_t s);
sbc_status launch_contract_16_24_32(int32_t M, bool bf16, const TileContractArgs &a, hipStream_t s);
sbc_status launch_dw(int32_t M, bool bf16, const TileDwArgs &a, hipStream_t s);

}  // namespace sbc
