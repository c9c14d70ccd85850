// tile_contract_kernel for the basis sizes of the point and fixed-decay event
// bases (M = 4, 8, 10).
#include "tile_launch.hpp"

namespace sbc {

template <int M, StageKind kKind>
static void launch_p(bool bf16, const TileContractArgs &a, hipStream_t s) {
    if (a.tall) {
        if (bf16) launch_contract<M, true, kKind, true>(a, s);
        else launch_contract<M, false, kKind, true>(a, s);
    } else {
        if (bf16) launch_contract<M, true, kKind, false>(a, s);
        else launch_contract<M, false, kKind, false>(a, s);
    }
}

template <int M>
static void launch_m(bool bf16, const TileContractArgs &a, hipStream_t s) {
    const StageKind kind = stage_kind(M, a.mode);
    if constexpr (M == 8 || M == 10) {
        if (kind == kCompact) {
            launch_p<M, kCompact>(bf16, a, s);
            return;
        }
    }
    if constexpr (M == 8) {
        if (kind == kEvents) {
            launch_p<M, kEvents>(bf16, a, s);
            return;
        }
    }
    launch_p<M, kValues>(bf16, a, s);
}

sbc_status launch_contract_4_8_10(int32_t M, bool bf16, const TileContractArgs &a, hipStream_t s) {
    if (M == 4) launch_m<4>(bf16, a, s);
    else if (M == 8) launch_m<8>(bf16, a, s);
    else launch_m<10>(bf16, a, s);
    SBC_LAUNCH_CHECK();
    return SBC_OK;
}

}  // namespace sbc
