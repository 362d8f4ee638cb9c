// z4c_variants_p4.hip -- instantiations of the tile kernels (see z4c_stage.h).
#include "z4c_cons.h"
#include "z4c_stage.h"

namespace z4c {

hipError_t launch_p4(int mode, int arith, const StageArgs &a, hipStream_t s)
{
    if (mode == MODE_CONS)
        return launch_cons<4, 2>(a, s);
    // FP32 at three waves per SIMD: 164 registers suffice without scratch and with
    // 26 of 27 slots three workgroups' LDS fits a CU (stage of 512 blocks of 16^3
    // with matter 0.891 ms, at two waves 0.946, FP64 0.948).
    return arith == Z4C_ARITH_FP32 ? launch_variant<4, 3, float>(mode, a, s)
                                   : launch_variant<4, 2, double>(mode, a, s);
}

}  // namespace z4c
