// bf16 instantiations of the blocked weight gradient.
#include "conv_wgrad_tile.h"

namespace dc {

hipError_t launch_wgrad_tile_bf16(const WgradArgs& a, hipStream_t s) {
#define X(id, now, ncw, wo, wc, wt, wk, tw) \
    if (a.tcfg == id) return launch_wgrad_tile<1, now, ncw, wo, wc, wt, wk, tw, wt_pixels(1, id), 1>(a, s);
    DC_WT_CONFIGS(X)
#undef X
    return hipErrorInvalidValue;
}

}  // namespace dc
