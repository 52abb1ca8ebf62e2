// Instantiations of the 1D step and run kernels for the P_F32 arithmetic mode.
#include "run1d.h"

namespace hweno {

hipError_t launch_step1d_f32(int flux, int cells, const Step1Args& a, int grid, hipStream_t s) {
    return step1d_launch_prec<P_F32>(flux, cells, a, grid, s);
}

hipError_t launch_run1d_f32(int flux, int waves, int nprob, const Run1Args& a, hipStream_t s) {
    return run1d_launch_prec<P_F32>(flux, waves, nprob, a, s);
}

}  // namespace hweno
