// Launcher of the 1D step kernel (instantiations live in step1d_<mode>.hip).
#include "internal.h"

namespace hweno {

hipError_t launch_step1d_f64(int flux, int cells, const Step1Args& a, int grid, hipStream_t s);
hipError_t launch_step1d_f32(int flux, int cells, const Step1Args& a, int grid, hipStream_t s);
hipError_t launch_step1d_acc64(int flux, int cells, const Step1Args& a, int grid, hipStream_t s);
hipError_t launch_step1d_kahan(int flux, int cells, const Step1Args& a, int grid, hipStream_t s);

// One cell per lane while the waves leave most of the GPU idle: the three
// stages are one serial chain, 3.5 us for one cell of a lane and 3 us more for
// a second (a step of 4000 cells, F64: 10.9 us with one, 13.9 with two); from
// some 30 000 cells the halo of 12 in 64 costs more than it (50 000 cells:
// 21.5 against 18.7 us, 4 million: 302 against 265).
int step1d_cells(const hweno_problem* probs, int32_t nprob, const hweno_config&) {
    int64_t waves = 0;
    for (int p = 0; p < nprob; ++p) waves += tiles_1d(probs[p].nx, 1);
    return waves <= 600 ? 1 : 2;
}

hipError_t launch_step1d(int prec, int flux, int cells, const Step1Args& a, int grid,
                         hipStream_t s) {
    if (a.ntiles <= 0) return hipSuccess;
    if (grid <= 0 || grid > a.ntiles) grid = a.ntiles;
    if (prec == P_F64) return launch_step1d_f64(flux, cells, a, grid, s);
    if (prec == P_F32) return launch_step1d_f32(flux, cells, a, grid, s);
    if (prec == P_ACC64) return launch_step1d_acc64(flux, cells, a, grid, s);
    if (prec == P_KAHAN) return launch_step1d_kahan(flux, cells, a, grid, s);
    return hipErrorInvalidValue;
}

}  // namespace hweno
