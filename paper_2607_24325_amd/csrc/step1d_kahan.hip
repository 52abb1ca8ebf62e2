// Instantiations of the 1D step kernel for the P_KAHAN arithmetic mode.
#include "step1d.h"

namespace hweno {

hipError_t launch_step1d_kahan(int flux, int cells, const Step1Args& a, int grid, hipStream_t s) {
    return step1d_launch_prec<P_KAHAN>(flux, cells, a, grid, s);
}

}  // namespace hweno
