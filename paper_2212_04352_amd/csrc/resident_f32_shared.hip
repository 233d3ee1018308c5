// resident_f32_shared.hip -- kernels of the configurations with both spin blocks of a trajectory in one workgroup, FP32.
#include "rk4_resident.h"

namespace ftwa {

const Config kConfigsF32Shared[] = {
    FTWA_RES_CFG(float, FTWA_F32, 2, 64, 16, 1, 1, 1, 1),
    FTWA_RES_CFG(float, FTWA_F32, 2, 128, 8, 2, 2, 2, 2),
    FTWA_RES_CFG(float, FTWA_F32, 2, 256, 4, 3, 3, 3, 3),
    FTWA_RES_CFG(float, FTWA_F32, 2, 512, 1, 5, 5, 5, 5),
    FTWA_RES_CFG(float, FTWA_F32, 2, 128, 8, 2, 2, 1, 1),
    FTWA_RES_CFG(float, FTWA_F32, 2, 256, 4, 3, 3, 1, 1),
    FTWA_RES_CFG(float, FTWA_F32, 2, 512, 1, 5, 5, 1, 1),
    FTWA_RES_CFG(float, FTWA_F32, 2, 64, 8, 1, 1, 1, 1),
    FTWA_RES_CFG(float, FTWA_F32, 2, 64, 4, 1, 1, 1, 1),
    FTWA_RES_CFG(float, FTWA_F32, 2, 64, 2, 1, 1, 1, 1),
    FTWA_RES_CFG(float, FTWA_F32, 2, 64, 1, 1, 1, 1, 1),
    FTWA_RES_CFG(float, FTWA_F32, 2, 128, 1, 2, 2, 1, 1),
    FTWA_RES_CFG(float, FTWA_F32, 2, 256, 1, 3, 3, 1, 1),
};

}  // namespace ftwa
