// z4c_variants_mon.hip -- instantiations of the stage kernel with the
// constraint monitor (FP64 arithmetic; see z4c_stage.h).
#include "z4c_stage.h"

namespace z4c {

hipError_t launch_monitor(int fd_order, const StageArgs &a, hipStream_t s)
{
    return fd_order == 6 ? launch_kernel<6, 2, double, MODE_RK, true>(a, s)
                         : launch_kernel<4, 2, double, MODE_RK, true>(a, s);
}

}  // namespace z4c
