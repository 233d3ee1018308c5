// evolve_shared_f32.hip -- the shared-pack resident kernels in FP32.
#include "evolve_shared.h"

namespace ftwa {

const SharedShape kSharedF32[kSharedShapes] = {
    FTWA_SHARED(float, FTWA_F32, 1, 1, 64, 1, false, false),
    FTWA_SHARED(float, FTWA_F32, 1, 2, 512, 1, false, false),
    FTWA_SHARED(float, FTWA_F32, 2, 2, 768, 1, false, false),
    FTWA_SHARED(float, FTWA_F32, 3, 2, 512, 1, true, false),
    FTWA_SHARED(float, FTWA_F32, 3, 2, 768, 1, false, true),
    FTWA_SHARED(float, FTWA_F32, 5, 2, 512, 1, false, true),
};

}  // namespace ftwa
