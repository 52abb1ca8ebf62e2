// Launchers of the 1D step and run kernels (instantiations live in
// step1d_<mode>.hip) and the rules that choose between them.
#include "internal.h"

namespace hweno {

hipError_t launch_step1d_f64(int flux, int cells, const Step1Args& a, int grid, hipStream_t s);
hipError_t launch_step1d_f32(int flux, int cells, const Step1Args& a, int grid, hipStream_t s);
hipError_t launch_step1d_acc64(int flux, int cells, const Step1Args& a, int grid, hipStream_t s);
hipError_t launch_step1d_kahan(int flux, int cells, const Step1Args& a, int grid, hipStream_t s);

hipError_t launch_run1d_f64(int flux, int waves, int nprob, const Run1Args& a, hipStream_t s);
hipError_t launch_run1d_f32(int flux, int waves, int nprob, const Run1Args& a, hipStream_t s);
hipError_t launch_run1d_acc64(int flux, int waves, int nprob, const Run1Args& a, hipStream_t s);
hipError_t launch_run1d_kahan(int flux, int waves, int nprob, const Run1Args& a, hipStream_t s);

// One cell per lane while the waves leave most of the GPU idle: the three
// stages are one serial chain, 3.5 us for one cell of a lane and 2.5 us more for
// a second (a step of 4000 cells, F64: 10.5 us with one, 13.1 with two);
// between 130 000 and 200 000 cells the halo of 12 in 64 comes to cost more than
// that (130 000: 17.0 against 19.7 us, 200 000: 21.2 against 20.8, 4 million: 277
// against 246).
int step1d_cells(const hweno_problem* probs, int32_t nprob) {
    int64_t waves = 0;
    for (int p = 0; p < nprob; ++p) waves += tiles_1d(probs[p].nx, 1);
    return waves <= 2500 ? 1 : 2;
}

// A problem that fits a workgroup's eight waves (two to a SIMD of its CU) is
// stepped there whatever the number of problems: a step of one problem of 416
// cells takes 8 us instead of 10 with the step kernel (characteristic 9.6 instead
// of 10.7), of 4096 such problems 132 instead of 141 (160 instead of 162), of
// 4096 of 20 cells 45 instead of 54, in F64.  Every workgroup has the waves of the
// largest problem: 4096 problems of 20 cells beside one of 416 take 83 us, 48 with
// the step kernel.
int run1d_waves(const hweno_problem* probs, int32_t nprob, const hweno_config& cfg) {
    if (cfg.alpha_stage) return 0;
    int most = 0;
    for (int p = 0; p < nprob; ++p) {
        const int w = tiles_1d(probs[p].nx, 1);
        most = w > most ? w : most;
    }
    return most <= RUN1D_WAVES ? most : 0;
}

// 4096 steps of as many problems as there are CUs, proportionally fewer of more,
// so that a launch ends within some 50 ms (5 to 12 us a step and such round): the
// work of other streams and a reader of the results wait no longer for it.
int run1d_steps(int nprob) {
    const int rounds = (nprob + 255) / 256;
    return rounds < 4096 ? 4096 / rounds : 1;
}

hipError_t launch_run1d(int prec, int flux, int waves, int nprob, const Run1Args& a,
                        hipStream_t s) {
    if (waves < 1 || waves > RUN1D_WAVES || nprob < 1) return hipErrorInvalidValue;
    if (prec == P_F64) return launch_run1d_f64(flux, waves, nprob, a, s);
    if (prec == P_F32) return launch_run1d_f32(flux, waves, nprob, a, s);
    if (prec == P_ACC64) return launch_run1d_acc64(flux, waves, nprob, a, s);
    if (prec == P_KAHAN) return launch_run1d_kahan(flux, waves, nprob, a, s);
    return hipErrorInvalidValue;
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
