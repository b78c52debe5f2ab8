// pdmi_step_staged_f32.hip -- launcher of the staged-mapping step kernels, FP32 bond arithmetic.
#include "pdmi_step.h"

namespace pdmi {

hipError_t launch_step_staged_f32(const StepArgs& a, int mode, bool ext, hipStream_t s)
{
    if (a.ntiles <= 0) return hipSuccess;
    return ext ? launch_staged_n<true, true>(a, mode, s) : launch_staged_n<true, false>(a, mode, s);
}

}  // namespace pdmi
