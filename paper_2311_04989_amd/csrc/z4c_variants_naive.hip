// z4c_variants_naive.hip -- instantiations of the naive-FP32 right-hand side
// (see z4c_stage.h): every staged sample rounded to float before the stencil
// differences, order 6.
#include "z4c_stage.h"

namespace z4c {

hipError_t launch_naive(const StageArgs &a, hipStream_t s)
{
    return launch_kernel<6, 2, float, MODE_RHS, false, false, true>(a, s);
}

}  // namespace z4c
