// resident_f64_shared.hip -- kernels of the configurations with both spin blocks of a trajectory in one workgroup, FP64.
#include "rk4_resident.h"

namespace ftwa {

const Config kConfigsF64Shared[] = {
    FTWA_RES_CFG(double, FTWA_F64, 2, 64, 16, 1, 1, 1, 1),
    FTWA_RES_CFG(double, FTWA_F64, 2, 128, 8, 2, 2, 2, 2),
    FTWA_RES_CFG(double, FTWA_F64, 2, 256, 3, 3, 3, 3, 3),
    FTWA_RES_CFG(double, FTWA_F64, 2, 512, 1, 5, 5, 5, 5),
    FTWA_RES_CFG(double, FTWA_F64, 2, 128, 8, 2, 2, 1, 1),
    FTWA_RES_CFG(double, FTWA_F64, 2, 256, 3, 3, 3, 1, 1),
    FTWA_RES_CFG(double, FTWA_F64, 2, 512, 1, 5, 5, 1, 1),
    FTWA_RES_CFG(double, FTWA_F64, 2, 384, 2, 2, 2, 1, 1),
    FTWA_RES_CFG(double, FTWA_F64, 2, 384, 2, 2, 2, 2, 2),
    FTWA_RES_CFG(double, FTWA_F64, 2, 64, 8, 1, 1, 1, 1),
    FTWA_RES_CFG(double, FTWA_F64, 2, 64, 4, 1, 1, 1, 1),
    FTWA_RES_CFG(double, FTWA_F64, 2, 64, 2, 1, 1, 1, 1),
    FTWA_RES_CFG(double, FTWA_F64, 2, 64, 1, 1, 1, 1, 1),
    FTWA_RES_CFG(double, FTWA_F64, 2, 128, 1, 2, 2, 1, 1),
    FTWA_RES_CFG(double, FTWA_F64, 2, 384, 1, 2, 2, 1, 1),
};

}  // namespace ftwa
