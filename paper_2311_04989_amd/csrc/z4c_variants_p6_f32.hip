// z4c_variants_p6_f32.hip -- instantiations of the tile kernels (see z4c_stage.h).
#include "z4c_stage.h"

namespace z4c {

hipError_t launch_p6_f32(int mode, const StageArgs &a, hipStream_t s)
{
    // Two waves per SIMD: at three, 168 registers spill 20 to 35 values and
    // the RK4 step of 8 x 64^3 blocks takes 4.43 ms against 4.07 ms.
    return launch_variant<6, 2, float>(mode, a, s);
}

}  // namespace z4c
