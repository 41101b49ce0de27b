// bf16 instantiations of the blocked implicit GEMM over the four output
// phases of a stride-2 backward-data.
#include "conv_igemm_tile.h"

namespace dc {

#define DC_TILE_CFGS(X) X(1, 2, 1, 1, 4) X(2, 1, 1, 2, 2) X(5, 1, 1, 1, 4)

hipError_t launch_tile_bf16_bp(const IgemmArgs& a, hipStream_t s) {
#define X(id, nob, npb, wo, wp) \
    if (a.tcfg == id) { \
        constexpr int OB = 32 * nob * wo; \
        if (a.tkg == 2 && a.twm == kWBlocks && a.tccg == 4) return launch_tile<1, 4, nob, npb, wo, wp, kWBlocks, 1, OB == 32 ? 1 : 2, 1, true, 2>(a, s); \
        if (a.tkg != 1) return hipErrorInvalidValue; \
        if (a.twm == kWBlocks && a.tccg == 2) return launch_tile<1, 2, nob, npb, wo, wp, kWBlocks, 1, 2, 1, true>(a, s); \
        if (a.twm == kWBlocks && a.tccg == 4) return launch_tile<1, 4, nob, npb, wo, wp, kWBlocks, 1, OB == 32 ? 1 : 2, 1, true>(a, s); \
        if (a.twm == kWBlocks && a.tccg == 8) return launch_tile<1, 8, nob, npb, wo, wp, kWBlocks, 1, 1, 1, true>(a, s); \
        if (a.twm == kWGather && a.tccg == 2) return launch_tile<1, 2, nob, npb, wo, wp, kWGather, 1, 5, 1, true>(a, s); \
        if (a.twm == kWGather && a.tccg == 4) return launch_tile<1, 4, nob, npb, wo, wp, kWGather, 1, 5, 1, true>(a, s); \
        if (a.twm == kWGather && a.tccg == 8) return launch_tile<1, 8, nob, npb, wo, wp, kWGather, 1, 2, 1, true>(a, s); \
    }
    DC_TILE_CFGS(X)
#undef X
    return hipErrorInvalidValue;
}

}  // namespace dc
