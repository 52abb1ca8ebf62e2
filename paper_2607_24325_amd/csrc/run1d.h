// Many SSP-RK3 steps of small 1D problems in one launch: a workgroup holds a
// whole problem in LDS and takes step after step, until the steps asked for
// are taken or the problem is at its end.
//
// A step of a small problem is a short serial chain (three stages of one cell,
// about 4 us in FP64), to which a launch per step adds 7 us: the gap between
// launches, the loads of table and state, the stores and the atomics that end
// the step.  Here waves cover the problem as in the step kernel (52 cells each,
// six halo cells a side, read from LDS); between steps the workgroup exchanges
// the new cells and the wave maxima of their speeds through LDS, two barriers.
// Each problem fits one workgroup of at most RUN1D_WAVES waves, so nothing ever
// waits for another workgroup.  The first step's speeds are reduced here too,
// with the arithmetic of every other kernel.
#pragma once

#include "step1d.h"

namespace hweno {

template <int P, int K, int FLUX, bool CH>
__global__ void __launch_bounds__(64 * RUN1D_WAVES) run1d_kernel(Run1Args a) {
    using TU = typename PrecT<P>::TU;
    using TD = typename PrecT<P>::TD;
    using T = typename PrecT<P>::T;
    using TA = typename PrecT<P>::TA;
    constexpr int OUT = 64 - STEP1D_HALO;
    constexpr int NMAX = RUN1D_WAVES * OUT;
    __shared__ TU su[K][NMAX];           // the problem's state
    __shared__ TD sv[K][NMAX];
    __shared__ TU gu[RUN1D_WAVES][K][64];   // per wave: ghost refill
    __shared__ TD gv[RUN1D_WAVES][K][64];
    __shared__ double s_mx[RUN1D_WAVES];
    __shared__ long long s_bad[RUN1D_WAVES];

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), nwave = blockDim.x >> 6;
    const Scheme& sch = a.sch;
    const int p = blockIdx.x;
    const bool ext = a.ext_in != nullptr;   // one problem, its state in the caller's arrays
    ProbDev Q = ext ? a.prob : a.probs[p];
    const int nx = Q.nx, bcx = Q.bc_x;
    TU* Gu = (TU*)(Q.cur ? a.s[1].u : a.s[0].u) + Q.off_u;
    TD* Gv = (TD*)(Q.cur ? a.s[1].d : a.s[0].d) + Q.off_d;
    for (int k = tid; k < nx; k += blockDim.x)
#pragma unroll
        for (int c = 0; c < K; ++c) {
            su[c][k] = ext ? (TU)a.ext_in[(int64_t)c * nx + k] : Gu[(int64_t)c * nx + k];
            sv[c][k] = ext ? (TD)a.ext_in[(int64_t)(K + c) * nx + k] : Gv[(int64_t)c * nx + k];
        }
    __syncthreads();

    const int k = wave * OUT - 6 + lane;    // this lane's cell, and whether it is written
    const bool emit = lane >= 6 && lane < 6 + OUT && k < nx;
    // Speeds of the cells written: the waves' maxima and first non-admissible
    // cells into LDS, then to every thread after a barrier.
    auto reduce_wave = [&](const double* w) {
        double mx = 0.0, sy;
        long long bad = LLONG_MAX;
        if (emit) {
            double sx;
            if (wave_speed<FLUX, 1, K>(w, sch, sx, sy)) mx = sx;
            else bad = k;
        }
        mx = wave_max_d(mx);
        if (__any(bad != LLONG_MAX)) bad = wave_min_ll(bad);
        if (lane == 0) {
            s_mx[wave] = mx;
            s_bad[wave] = bad;
        }
    };
    auto take_speeds = [&]() {
        double mx = s_mx[0];
        long long bad = s_bad[0];
        for (int v = 1; v < nwave; ++v) {
            mx = fmax(mx, s_mx[v]);
            bad = s_bad[v] < bad ? s_bad[v] : bad;
        }
        Q.ax_bits = (uint64_t)__double_as_longlong(mx);
        if (bad != LLONG_MAX) {
            Q.bad_cell = bad < Q.bad_cell ? bad : Q.bad_cell;
            Q.err |= ERR_STATE_BAD;
        }
    };
    if (Q.t < Q.t_end && !Q.err && !Q.alpha_valid) {
        double w[K];
#pragma unroll
        for (int c = 0; c < K; ++c) w[c] = emit ? (double)su[c][k] : 0.0;
        reduce_wave(w);
        __syncthreads();
        take_speeds();
        __syncthreads();   // the maxima are written again by the first step
    }

    int taken = 0;
    for (int s = 0; s < a.nsteps; ++s) {
        const StepChoice step = choose_step(Q, a.cfl, 1, a.flags);
        Q.active = step.act;
        Q.last = step.last;
        Q.dt = step.dt;
        if (!step.act) break;   // the same for every thread
        ++taken;
        TU u[K][1];
        TD v[K][1];
        if (wave * OUT < nx) {
            const int src = bc_map(k, nx, bcx);
            const bool mir = FLUX == F_EULER && wall_mirrored(k, nx, bcx);
#pragma unroll
            for (int c = 0; c < K; ++c) {
                u[c][0] = neg_if(su[c][src], mir && c == 1);
                v[c][0] = neg_if(sv[c][src], mir && c != 1);
            }
            const Wave1D<T, TA> w = wave1d<T, TA>(Q, step.dt, wave * OUT - 6, 64);
            advance1d<P, K, FLUX, CH, 1>(u, v, w, sch, gu[wave], gv[wave]);
        } else {
#pragma unroll
            for (int c = 0; c < K; ++c) u[c][0] = (TU)0, v[c][0] = (TD)0;
        }
        double w[K];
#pragma unroll
        for (int c = 0; c < K; ++c) w[c] = (double)u[c][0];
        reduce_wave(w);
        __syncthreads();   // every wave has read the old cells; maxima are ready
        if (emit)
#pragma unroll
            for (int c = 0; c < K; ++c) {
                su[c][k] = u[c][0];
                sv[c][k] = v[c][0];
            }
        take_speeds();
        Q.alpha_valid = 1;
        Q.t = step.last ? Q.t_end : Q.t + step.dt;
        __syncthreads();   // the new cells are ready, the maxima read
    }

    for (int c = 0; c < K; ++c)
        for (int i = tid; i < nx; i += blockDim.x) {
            if (ext) {
                a.ext_out[(int64_t)c * nx + i] = (double)su[c][i];
                a.ext_out[(int64_t)(K + c) * nx + i] = (double)sv[c][i];
            } else if (taken) {
                Gu[(int64_t)c * nx + i] = su[c][i];
                Gv[(int64_t)c * nx + i] = sv[c][i];
            }
        }
    if (tid != 0) return;
    if (ext) {
        if (a.dt_out) *a.dt_out = Q.active && !Q.err ? Q.dt : 0.0;
        if (a.bad_out) *a.bad_out = Q.err ? Q.bad_cell : -1;
        return;
    }
    ProbDev& G = a.probs[p];
    G.t = Q.t;
    G.dt = Q.dt;
    G.ax_bits = Q.ax_bits;
    G.ay_bits = 0;
    G.active = Q.active;
    G.last = Q.last;
    G.err = Q.err;
    G.alpha_valid = Q.alpha_valid;
    G.bad_cell = Q.bad_cell;
    end_problem(p, Q.t < Q.t_end && !Q.err, taken, a.ctl);
}

template <int P>
hipError_t run1d_launch_prec(int flux, int waves, int nprob, const Run1Args& a, hipStream_t s) {
    const int threads = 64 * waves;
    if (flux == F_ADV) run1d_kernel<P, 1, F_ADV, false><<<nprob, threads, 0, s>>>(a);
    else if (flux == F_BURGERS) run1d_kernel<P, 1, F_BURGERS, false><<<nprob, threads, 0, s>>>(a);
    else if (a.sch.charwise) run1d_kernel<P, 3, F_EULER, true><<<nprob, threads, 0, s>>>(a);
    else run1d_kernel<P, 3, F_EULER, false><<<nprob, threads, 0, s>>>(a);
    return hipGetLastError();
}

}  // namespace hweno
