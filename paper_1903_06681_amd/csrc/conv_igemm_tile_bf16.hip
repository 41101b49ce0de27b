// bf16 instantiations of the blocked implicit GEMM (one output phase).
#include "conv_igemm_tile.h"

namespace dc {

// (MFMA tiles per wave, waves): OB x PT = 64x256, 64x128, 64x64, 32x256, 128x128
#define DC_TILE_CFGS(X) X(0, 2, 2, 1, 4) X(1, 2, 1, 1, 4) X(2, 1, 1, 2, 2) X(3, 1, 2, 1, 4) X(4, 2, 2, 2, 2)

hipError_t launch_tile_bf16(const IgemmArgs& a, hipStream_t s) {
    const int T = a.R * a.S;
#define X(id, nob, npb, wo, wp) \
    if (a.tcfg == id) { \
        constexpr int OB = 32 * nob * wo; \
        if constexpr (id >= 1 && id <= 3) { \
            if (a.tkg == 2 && a.twm == kWRows && T == 9 && a.tccg == 4) return launch_tile<1, 4, nob, npb, wo, wp, kWRows, 9, (OB + 63) / 64, 1, false, 2>(a, s); \
            if (a.tkg == 2 && a.twm == kWBlocks && a.tccg == 4) return launch_tile<1, 4, nob, npb, wo, wp, kWBlocks, 1, OB == 32 ? 1 : 2, 1, false, 2>(a, s); \
        } \
        if (a.tkg != 1) return hipErrorInvalidValue; \
        if (a.twm == kWRows && T == 9 && a.tccg == 4) return launch_tile<1, 4, nob, npb, wo, wp, kWRows, 9, (OB + 63) / 64, 2, false>(a, s); \
        if (a.twm == kWRows && T == 1 && a.tccg == 8) return launch_tile<1, 8, nob, npb, wo, wp, kWRows, 1, (OB + 31) / 32, 2, false>(a, s); \
        if (a.twm == kWBlocks && a.tccg == 2) return launch_tile<1, 2, nob, npb, wo, wp, kWBlocks, 1, 2, 1, false>(a, s); \
        if (a.twm == kWBlocks && a.tccg == 4) return launch_tile<1, 4, nob, npb, wo, wp, kWBlocks, 1, (OB + 32) / 64 + (OB > 32 ? 1 : 0), 2, false>(a, s); \
        if (a.twm == kWBlocks && a.tccg == 8) return launch_tile<1, 8, nob, npb, wo, wp, kWBlocks, 1, 1, 2, false>(a, s); \
        if constexpr (id >= 1 && id <= 3) { \
            if (a.twm == kWGather && a.tccg == 2) return launch_tile<1, 2, nob, npb, wo, wp, kWGather, 1, OB == 32 ? 5 : 9, 1, false>(a, s); \
            if (a.twm == kWGather && a.tccg == 4) return launch_tile<1, 4, nob, npb, wo, wp, kWGather, 1, OB == 32 ? 5 : 9, 1, false>(a, s); \
            if (a.twm == kWGather && a.tccg == 8) return launch_tile<1, 8, nob, npb, wo, wp, kWGather, 1, OB == 32 ? 1 : 2, 2, false>(a, s); \
        } \
    }
    DC_TILE_CFGS(X)
#undef X
    return hipErrorInvalidValue;
}

}  // namespace dc
