// z4c_variants_p4.hip -- instantiations of the tile kernels (see z4c_stage.h).
#include "z4c_cons.h"
#include "z4c_stage.h"

namespace z4c {

hipError_t launch_p4(int mode, int arith, const StageArgs &a, hipStream_t s)
{
    if (mode == MODE_CONS)
        return launch_cons<4, 2>(a, s);
    return arith == Z4C_ARITH_FP32 ? launch_variant<4, 3, float>(mode, a, s)
                                   : launch_variant<4, 2, double>(mode, a, s);
}

}  // namespace z4c
