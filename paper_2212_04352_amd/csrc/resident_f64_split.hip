// resident_f64_split.hip -- kernels of the configurations with an FP64 spin block over several workgroups.
#include "rk4_split.h"

namespace ftwa {

const Config kConfigsF64Split[] = {
    // (the last: three waves per SIMD, 12 % faster than 512 threads at N = 150;
    // at three and four parts the extra waves spill)
    FTWA_SPLIT_CFG(double, FTWA_F64, 2, 512, 6, 6, 4, 1, 2, 1, 2, 1, true),
    FTWA_SPLIT_CFG(double, FTWA_F64, 3, 512, 7, 7, 4, 1, 1, 2, 4, 2, true),
    FTWA_SPLIT_CFG(double, FTWA_F64, 4, 512, 5, 5, 2, 1, 1, 1, 4, 3, true),
    FTWA_SPLIT_CFG(double, FTWA_F64, 2, 768, 4, 4, 3, 1, 1, 1, 2, 1, true),
};

}  // namespace ftwa
