// fp32 instantiations of the blocked weight gradient (three bf16 parts a value).
#include "conv_wgrad_tile.h"

namespace dc {

hipError_t launch_wgrad_tile_f32(const WgradArgs& a, hipStream_t s) {
#define X(id, now, ncw, wo, wc, wt, wk, tw) \
    if constexpr (id <= 5 || id == 7) { \
        if (a.tcfg == id) return launch_wgrad_tile<3, now, ncw, wo, wc, wt, wk, tw, wt_pixels(3, id), 1>(a, s); \
    }
    DC_WT_CONFIGS(X)
#undef X
    return hipErrorInvalidValue;
}

}  // namespace dc
