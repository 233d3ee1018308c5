// resident_f32_spin.hip -- kernels of the configurations with one FP32 spin block per workgroup.
#include "rk4_resident.h"

namespace ftwa {

const Config kConfigsF32Spin[] = {
    FTWA_RES_CFG(float, FTWA_F32, 1, 768, 1, 8, 8, 2, 2),
    FTWA_RES_CFG(float, FTWA_F32, 1, 768, 1, 13, 13, 2, 2),
    FTWA_RES_CFG(float, FTWA_F32, 1, 1024, 1, 10, 10, 2, 2),
    FTWA_RES_CFG(float, FTWA_F32, 1, 512, 1, 20, 20, 2, 2),
    FTWA_RES_CFG(float, FTWA_F32, 1, 768, 1, 13, 13, 13, 13),
};

}  // namespace ftwa
