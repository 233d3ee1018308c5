// resident_f64_split.hip -- kernels of the configurations with an FP64 spin block over several workgroups.
#include "rk4_split.h"

namespace ftwa {

const Config kConfigsF64Split[] = {
    // Two parts of 512 threads: 150 sites 7.2 ms where the 768-thread form,
    // which spills, takes 7.8 (500 trajectories, 50 steps); that one holds
    // lattices with more boundary elements (112-site torus 4.6 ms, three parts
    // 8.3).  The last: up to about 110 sites (8.2 -> 6.6 ms at 110, 1024
    // trajectories, 30 steps).
    FTWA_SPLIT_CFG(double, FTWA_F64, 2, 512, 6, 6, 4, 1, 2, 1, 2, 1, true),
    FTWA_SPLIT_CFG(double, FTWA_F64, 3, 512, 7, 7, 4, 1, 1, 2, 4, 3, true),
    FTWA_SPLIT_CFG(double, FTWA_F64, 4, 512, 5, 5, 2, 1, 1, 1, 4, 3, true),
    FTWA_SPLIT_CFG(double, FTWA_F64, 2, 768, 4, 4, 3, 1, 1, 1, 2, 1, true),
    FTWA_SPLIT_CFG(double, FTWA_F64, 2, 512, 4, 4, 3, 1, 1, 1, 2, 1, true),
};

}  // namespace ftwa
