// tile_contract_kernel for the learned-decay event basis (M = 16, 24, 32).
#include "tile_launch.hpp"

namespace sbc {

template <int M>
static void launch_m(bool bf16, const TileContractArgs &a, hipStream_t s) {
    if (stage_kind(M, a.mode) == kEvents) {
        if (bf16) launch_contract<M, true, kEvents, false>(a, s);
        else launch_contract<M, false, kEvents, false>(a, s);
    } else {
        if (bf16) launch_contract<M, true, kValues, false>(a, s);
        else launch_contract<M, false, kValues, false>(a, s);
    }
}

sbc_status launch_contract_16_24_32(int32_t M, bool bf16, const TileContractArgs &a,
                                    hipStream_t s) {
    if (M == 16) launch_m<16>(bf16, a, s);
    else if (M == 24) launch_m<24>(bf16, a, s);
    else launch_m<32>(bf16, a, s);
    SBC_LAUNCH_CHECK();
    return SBC_OK;
}

}  // namespace sbc
