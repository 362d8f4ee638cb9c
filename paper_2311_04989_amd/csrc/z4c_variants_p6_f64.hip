// z4c_variants_p6_f64.hip -- instantiations of the tile kernels (see z4c_stage.h).
#include "z4c_cons.h"
#include "z4c_stage.h"

namespace z4c {

hipError_t launch_p6_f64(int mode, const StageArgs &a, hipStream_t s)
{
    return mode == MODE_CONS ? launch_cons<6, 2>(a, s) : launch_variant<6, 2, double>(mode, a, s);
}

}  // namespace z4c
