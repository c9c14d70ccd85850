// tile_dw_kernel for every basis size.
#include "tile_launch.hpp"

namespace sbc {

template <int M, bool kXbf, StageKind kKind, int NPB>
static void launch_one(const TileDwArgs &a, hipStream_t s) {
    using T = DwShape<M, NPB, kKind>;
    const int32_t slices = (a.CQ + kTileCS - 1) / kTileCS;
    const int32_t chunks = (a.CP + 16 * NPB - 1) / (16 * NPB);
    hipLaunchKernelGGL((tile_dw_kernel<M, kXbf, kKind, NPB>),
                       dim3((unsigned)a.splits, (unsigned)(slices * chunks)), dim3(kTileThreads),
                       0, s, a.p, a.v, a.g, a.mode, a.P, a.CP, a.Q, a.CQ,
                       (a.p.n_rows + T::TR - 1) / T::TR, a.part);
}

// Registers: M = 32 spills 166 to 175 at one wave a SIMD (the weight gradient and
// the decay gradient of four decays), given values of 16 functions 28 to 36.  Shapes
// that lose by it go to the separate kernels (route_cost.hpp).
template <int M, StageKind kKind>
static void launch_p(bool bf16, const TileDwArgs &a, hipStream_t s) {
    if constexpr (M < 16) {
        if (dw_npb(M, a.CP) == 4) {
            if (bf16) launch_one<M, true, kKind, 4>(a, s);
            else launch_one<M, false, kKind, 4>(a, s);
            return;
        }
    }
    if (bf16) launch_one<M, true, kKind, 2>(a, s);
    else launch_one<M, false, kKind, 2>(a, s);
}

template <int M>
static void launch_m(bool bf16, const TileDwArgs &a, hipStream_t s) {
    const StageKind kind = stage_kind(M, a.mode);
    if constexpr (M == 8 || M == 10) {
        if (kind == kCompact) {
            launch_p<M, kCompact>(bf16, a, s);
            return;
        }
    }
    if constexpr (M % 8 == 0) {
        if (kind == kEvents) {
            launch_p<M, kEvents>(bf16, a, s);
            return;
        }
    }
    launch_p<M, kValues>(bf16, a, s);
}

sbc_status launch_dw(int32_t M, bool bf16, const TileDwArgs &a, hipStream_t s) {
    switch (M) {
        case 4: launch_m<4>(bf16, a, s); break;
        case 8: launch_m<8>(bf16, a, s); break;
        case 10: launch_m<10>(bf16, a, s); break;
        case 16: launch_m<16>(bf16, a, s); break;
        case 24: launch_m<24>(bf16, a, s); break;
        default: launch_m<32>(bf16, a, s); break;
    }
    SBC_LAUNCH_CHECK();
    return SBC_OK;
}

}  // namespace sbc
