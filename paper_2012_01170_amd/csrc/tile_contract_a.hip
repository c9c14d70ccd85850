// tile_contract_kernel for the basis sizes of the point and fixed-decay event
// bases (M = 4, 8, 10).
#include "tile_launch.hpp"

namespace sbc {

template <int M, bool kCompact>
static void launch_p(bool bf16, const TileContractArgs &a, hipStream_t s) {
    if (a.tr == 64) {
        if (bf16) launch_contract<M, true, kCompact, 64>(a, s);
        else launch_contract<M, false, kCompact, 64>(a, s);
    } else {
        if (bf16) launch_contract<M, true, kCompact, 32>(a, s);
        else launch_contract<M, false, kCompact, 32>(a, s);
    }
}

template <int M>
static void launch_m(bool bf16, const TileContractArgs &a, hipStream_t s) {
    if constexpr (M == 8 || M == 10) {
        if (a.mode == SBC_BASIS_MONO8 + 1 || a.mode == SBC_BASIS_WMONO10 + 1) {
            launch_p<M, true>(bf16, a, s);
            return;
        }
    }
    launch_p<M, false>(bf16, a, s);
}

sbc_status launch_contract_4_8_10(int32_t M, bool bf16, const TileContractArgs &a, hipStream_t s) {
    if (M == 4) launch_m<4>(bf16, a, s);
    else if (M == 8) launch_m<8>(bf16, a, s);
    else launch_m<10>(bf16, a, s);
    SBC_LAUNCH_CHECK();
    return SBC_OK;
}

}  // namespace sbc
