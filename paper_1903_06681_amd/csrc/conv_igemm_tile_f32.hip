// fp32 instantiations of the blocked implicit GEMM (three bf16 parts a value).
#include "conv_igemm_tile.h"

namespace dc {

hipError_t launch_tile_f32(const IgemmArgs& a, hipStream_t s) {
#define X(id, nob, npb, wo, wp, BPH) \
    if (a.tcfg == id && (a.bp != 0) == BPH) { \
        constexpr int OB = 32 * nob * wo; \
        if (a.tkg == 2 && a.tccg == 2) return launch_tile<3, 2, nob, npb, wo, wp, kWGather, 1, OB == 32 ? 3 : 5, 1, BPH, 2>(a, s); \
        if (a.tkg != 1) return hipErrorInvalidValue; \
        if constexpr (!BPH && id != 1) { \
            if (a.tsep && a.tccg == 2) return launch_tile<3, 2, nob, npb, wo, wp, kWGather, 1, OB == 32 ? 3 : 5, 2, false, 1, true>(a, s); \
            if (a.tsep && a.tccg == 4) return launch_tile<3, 4, nob, npb, wo, wp, kWGather, 1, 1, 2, false, 1, true>(a, s); \
        } \
        if (a.tsep) return hipErrorInvalidValue; \
        if (a.tccg == 2) return launch_tile<3, 2, nob, npb, wo, wp, kWGather, 1, OB == 32 ? 3 : 5, BPH ? 1 : 2, BPH>(a, s); \
        if (a.tccg == 4) return launch_tile<3, 4, nob, npb, wo, wp, kWGather, 1, 1, BPH ? 1 : 2, BPH>(a, s); \
    }
    X(1, 2, 1, 1, 4, false) X(2, 1, 1, 2, 2, false) X(3, 1, 2, 1, 4, false) X(5, 1, 1, 1, 4, false)
    X(2, 1, 1, 2, 2, true) X(5, 1, 1, 1, 4, true)
#undef X
    return hipErrorInvalidValue;
}

}  // namespace dc
