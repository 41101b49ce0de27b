// 3x3 instantiations of the rolling-row kernel with non-temporal stores.
#include "conv_igemm_roll.h"

namespace dc {

hipError_t launch_roll3_nt(const IgemmArgs& a, hipStream_t s) {
    switch (a.rows_per_seg % 3) {
        case 0: return launch_roll<2, 3, 3, 4, 0, true>(a, s);
        case 1: return launch_roll<2, 3, 3, 4, 1, true>(a, s);
        default: return launch_roll<2, 3, 3, 4, 2, true>(a, s);
    }
}

}  // namespace dc
