// evolve_shared_f64.hip -- the shared-pack resident kernels in FP64.
#include "evolve_shared.h"

namespace ftwa {

const SharedShape kSharedF64[kSharedShapes] = {
    FTWA_SHARED(double, FTWA_F64, 1, 1, 64, 1, false, false),
    FTWA_SHARED(double, FTWA_F64, 1, 1, 512, 1, false, false),
    FTWA_SHARED(double, FTWA_F64, 2, 1, 768, 1, false, false),
    FTWA_SHARED(double, FTWA_F64, 3, 1, 512, 1, false, false),
    FTWA_SHARED(double, FTWA_F64, 3, 1, 768, 1, false, true),
    FTWA_SHARED(double, FTWA_F64, 4, 1, 768, 1, false, true),
};

}  // namespace ftwa
