// 5x5 instantiations of the rolling-row kernel.
#include "conv_igemm_roll.h"

namespace dc {

hipError_t launch_roll5(const IgemmArgs& a, hipStream_t s) {
    switch (a.rows_per_seg % 5) {
        case 0: return launch_roll<1, 5, 5, 2, 0, false>(a, s);
        case 1: return launch_roll<1, 5, 5, 2, 1, false>(a, s);
        case 2: return launch_roll<1, 5, 5, 2, 2, false>(a, s);
        case 3: return launch_roll<1, 5, 5, 2, 3, false>(a, s);
        default: return launch_roll<1, 5, 5, 2, 4, false>(a, s);
    }
}

}  // namespace dc
