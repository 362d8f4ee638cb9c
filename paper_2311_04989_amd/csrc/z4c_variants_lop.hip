// z4c_variants_lop.hip -- instantiations of the right-hand side and stage
// kernels with lopsided advection (FP64 arithmetic; see z4c_stage.h).
#include "z4c_stage.h"

namespace z4c {

hipError_t launch_lopsided(int mode, int fd_order, const StageArgs &a, hipStream_t s)
{
    return fd_order == 6 ? launch_variant<6, 2, double, true>(mode, a, s)
                         : launch_variant<4, 2, double, true>(mode, a, s);
}

}  // namespace z4c
