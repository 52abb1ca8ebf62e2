// Per-step control kernels: wave-speed reduction for the global
// Lax-Friedrichs flux and the CFL rule, time-step selection, time update,
// and conversion between the boundary layout and the internal planes.
#include "device_common.h"

namespace hweno {

// Zeroes the wave-speed maxima that are about to be recomputed (SpeedSel)
// and, at the start of a step, the step counters.
__global__ void reset_kernel(ProbDev* probs, StepCtl* ctl, int nprob, int sel) {
    const int p = blockIdx.x * blockDim.x + threadIdx.x;
    if (p < nprob) {
        const ProbDev& P_ = probs[p];
        const bool pick = sel == SEL_ALL || (sel == SEL_STALE && !P_.alpha_valid) ||
                          (sel == SEL_ACTIVE && P_.active && !(P_.err & ERR_STAGE_BAD));
        if (pick) {
            probs[p].ax_bits = 0;
            probs[p].ay_bits = 0;
        }
    }
    if (p == 0 && sel != SEL_ACTIVE) {
        ctl->nactive = 0;
        ctl->step_active = 0;
    }
}

// alpha_x = max |f'(u)|, alpha_y = max |g'(u)| over the cell averages of a
// problem (Euler: |velocity| + sound speed), in double precision; cells that
// are not finite or have rho <= 0 / p <= 0 flag the problem.
template <int P, int FLUX, int DIM>
__global__ void __launch_bounds__(256) alpha_kernel(const void* u0, const void* u1, ProbDev* probs,
                                                    const Chunk* chunks, int nchunks,
                                                    Scheme sch, int sel) {
    using TU = typename PrecT<P>::TU;
    constexpr int K = FLUX == F_EULER ? (DIM == 1 ? 3 : 4) : 1;
    __shared__ double smx[4], smy[4];
    __shared__ long long sbad[4];
    for (int ch = blockIdx.x; ch < nchunks; ch += gridDim.x) {
        const Chunk chunk = chunks[ch];
        ProbDev& P_ = probs[chunk.prob];
        if (sel == SEL_STALE && (!(P_.t < P_.t_end) || P_.err || P_.alpha_valid)) continue;
        if (sel == SEL_ACTIVE && (!P_.active || (P_.err & ERR_STAGE_BAD))) continue;
        const int64_t plane = (int64_t)P_.nx * P_.ny;
        const TU* base = (const TU*)(P_.cur ? u1 : u0) + P_.off_u;
        double mx = 0.0, my = 0.0;
        long long bad = LLONG_MAX;
        // every load of the thread's cells first (lanes past the chunk read
        // its first cell), then the speeds
        constexpr int PER = CHUNK_CELLS / 256;
        double u[PER][K];
#pragma unroll
        for (int j = 0; j < PER; ++j) {
            const int k = threadIdx.x + 256 * j;
            const int64_t idx = chunk.start + (k < chunk.count ? k : 0);
#pragma unroll
            for (int c = 0; c < K; ++c) u[j][c] = (double)base[c * plane + idx];
        }
#pragma unroll
        for (int j = 0; j < PER; ++j) {
            const int k = threadIdx.x + 256 * j;
            if (k < chunk.count) {
                double sx, sy;
                if (wave_speed<FLUX, DIM, K>(u[j], sch, sx, sy)) {
                    mx = fmax(mx, sx);
                    my = fmax(my, sy);
                } else {
                    const int64_t idx = chunk.start + k;
                    if (idx < bad) bad = idx;
                }
            }
        }
        // thread 0 publishes the chunk's maxima; it reads the slots before
        // the reduction (lower bounds of their final values; see publish_max;
        // read at the start, when every block starts at once, they are mostly
        // still zero)
        uint64_t seen_x = 0, seen_y = 0;
        if (threadIdx.x == 0) {
            seen_x = peek_slot(&P_.ax_bits);
            seen_y = peek_slot(&P_.ay_bits);
        }
        mx = wave_max_d(mx);
        my = wave_max_d(my);
        if (__any(bad != LLONG_MAX)) bad = wave_min_ll(bad);
        const int wv = threadIdx.x >> 6;
        if ((threadIdx.x & 63) == 0) {
            smx[wv] = mx;
            smy[wv] = my;
            sbad[wv] = bad;
        }
        __syncthreads();
        if (threadIdx.x == 0) {
            for (int w = 1; w < 4; ++w) {
                mx = fmax(mx, smx[w]);
                my = fmax(my, smy[w]);
                bad = sbad[w] < bad ? sbad[w] : bad;
            }
            // non-negative doubles order like their bit patterns
            publish_max(&P_.ax_bits, mx, seen_x);
            publish_max(&P_.ay_bits, my, seen_y);
            if (bad != LLONG_MAX) {
                atomicMin((long long*)&P_.bad_cell, bad);
                atomicOr(&P_.err, sel == SEL_ACTIVE ? ERR_STAGE_BAD : ERR_STATE_BAD);
            }
        }
        __syncthreads();
    }
}

// Chooses a problem's step for kernels that read it from the table; returns
// whether the problem takes this step.
__device__ __forceinline__ int select_dt(ProbDev& P_, const StepCtl* ctl, int use_dt_in) {
    const StepChoice c = choose_step(P_, ctl, STEP_CHOOSE | (use_dt_in ? STEP_DT_IN : 0));
    P_.active = c.act;
    P_.last = c.last;
    P_.dt = c.dt;
    return c.act;
}

// own_ctl: the launch is one block that holds every problem and sets the
// step counters itself (no reset kernel before it); otherwise a reset kernel
// has cleared them and the blocks only raise step_active.
__global__ void dt_kernel(ProbDev* probs, StepCtl* ctl, int nprob, int use_dt_in, int own_ctl) {
    const int p = blockIdx.x * blockDim.x + threadIdx.x;
    const int act = p < nprob ? select_dt(probs[p], ctl, use_dt_in) : 0;
    if (own_ctl) {
        const int any = __syncthreads_or(act);
        if (threadIdx.x == 0) {
            ctl->nactive = 0;
            ctl->step_active = any;
        }
    } else if (act) {
        atomicOr(&ctl->step_active, 1);
    }
}

__device__ __forceinline__ void write_status(const ProbDev& P, ProbStatus* out) {
    *out = ProbStatus{P.t, as_double(P.ax_bits), as_double(P.ay_bits), P.bad_cell, P.err, P.nx};
}

// Converts between the boundary layout and the internal planes: blockIdx.y is
// the plane (var*K + comp), so that no element divides by the cell count.
// First thread of the launch: op.set_t, the problem's table entry for a new
// state; op.status, what the host asks of the table, into pinned host memory
// (the host waits for the launch before it reads it).
template <class TU, class TD, bool IN>
__global__ void __launch_bounds__(256) pack_kernel(const double* src, double* dst, TU* u0, TD* d0,
                                                   TU* u1, TD* d1, ProbDev* prob, int K,
                                                   int64_t ncell, PackOp op) {
    const int cur = prob->cur, plane = blockIdx.y;
    TU* u = (cur ? u1 : u0) + (int64_t)plane * ncell;
    TD* d = (cur ? d1 : d0) + (int64_t)(plane - K) * ncell;
    const int64_t e0 = (int64_t)plane * ncell;
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < ncell;
         i += (int64_t)gridDim.x * blockDim.x) {
        if (IN) {
            if (plane < K) u[i] = (TU)src[e0 + i];
            else d[i] = (TD)src[e0 + i];
        } else {
            dst[e0 + i] = plane < K ? (double)u[i] : (double)d[i];
        }
    }
    if (blockIdx.x != 0 || plane != 0 || threadIdx.x != 0) return;
    if (op.set_t) {
        prob->t = op.t;
        prob->err = 0;
        prob->err_next = 0;
        prob->bad_cell = INT64_MAX;
        prob->active = 0;
        prob->alpha_valid = 0;
    }
    if (op.status) write_status(*prob, op.status);
}

__global__ void status_kernel(const ProbDev* prob, ProbStatus* out) { write_status(*prob, out); }

// --------------------------------------------------------------- launchers

hipError_t launch_reset(ProbDev* probs, StepCtl* ctl, int nprob, int sel, hipStream_t s) {
    reset_kernel<<<(nprob + 255) / 256, 256, 0, s>>>(probs, ctl, nprob, sel);
    return hipGetLastError();
}

template <int P>
static hipError_t alpha_dispatch(int flux, int dim, const void* u0, const void* u1, ProbDev* probs,
                                 const Chunk* chunks, int nchunks, const Scheme& sch, int sel,
                                 int grid, hipStream_t s) {
    if (dim == 1) {
        if (flux == F_ADV) alpha_kernel<P, F_ADV, 1><<<grid, 256, 0, s>>>(u0, u1, probs, chunks, nchunks, sch, sel);
        else if (flux == F_BURGERS) alpha_kernel<P, F_BURGERS, 1><<<grid, 256, 0, s>>>(u0, u1, probs, chunks, nchunks, sch, sel);
        else alpha_kernel<P, F_EULER, 1><<<grid, 256, 0, s>>>(u0, u1, probs, chunks, nchunks, sch, sel);
    } else {
        if (flux == F_ADV) alpha_kernel<P, F_ADV, 2><<<grid, 256, 0, s>>>(u0, u1, probs, chunks, nchunks, sch, sel);
        else if (flux == F_BURGERS) alpha_kernel<P, F_BURGERS, 2><<<grid, 256, 0, s>>>(u0, u1, probs, chunks, nchunks, sch, sel);
        else alpha_kernel<P, F_EULER, 2><<<grid, 256, 0, s>>>(u0, u1, probs, chunks, nchunks, sch, sel);
    }
    return hipGetLastError();
}

hipError_t launch_alpha(int prec, int flux, int dim, const void* u0, const void* u1, ProbDev* probs,
                        const Chunk* chunks, int nchunks, const Scheme& sch, int sel,
                        int grid, hipStream_t s) {
    if (grid <= 0 || grid > nchunks) grid = nchunks;
    if (prec == P_F32) return alpha_dispatch<P_F32>(flux, dim, u0, u1, probs, chunks, nchunks, sch, sel, grid, s);
    if (prec == P_KAHAN) return alpha_dispatch<P_KAHAN>(flux, dim, u0, u1, probs, chunks, nchunks, sch, sel, grid, s);
    return alpha_dispatch<P_F64>(flux, dim, u0, u1, probs, chunks, nchunks, sch, sel, grid, s);
}

hipError_t launch_dt(ProbDev* probs, StepCtl* ctl, int nprob, int use_dt_in, int own_ctl,
                     hipStream_t s) {
    if (own_ctl && nprob > 256) return hipErrorInvalidValue;
    dt_kernel<<<(nprob + 255) / 256, 256, 0, s>>>(probs, ctl, nprob, use_dt_in, own_ctl);
    return hipGetLastError();
}

hipError_t launch_status(const ProbDev* prob, ProbStatus* out, hipStream_t s) {
    status_kernel<<<1, 1, 0, s>>>(prob, out);
    return hipGetLastError();
}

template <class TU, class TD>
static void pack_launch(const double* src, double* dst, StateBuf b0, StateBuf b1, ProbDev* prob,
                        int64_t off_u, int64_t off_d, int K, int nvar, int64_t ncell,
                        const PackOp& op, hipStream_t s) {
    const int64_t nb = (ncell + 255) / 256;
    const dim3 grid((unsigned)(nb < 8192 ? nb : 8192), (unsigned)(nvar * K));
    TU *u0 = (TU*)b0.u + off_u, *u1 = (TU*)b1.u + off_u;
    TD *d0 = (TD*)b0.d + off_d, *d1 = (TD*)b1.d + off_d;
    if (src) pack_kernel<TU, TD, true><<<grid, 256, 0, s>>>(src, dst, u0, d0, u1, d1, prob, K, ncell, op);
    else pack_kernel<TU, TD, false><<<grid, 256, 0, s>>>(src, dst, u0, d0, u1, d1, prob, K, ncell, op);
}

hipError_t launch_pack(int prec, const double* src, double* dst, StateBuf b0, StateBuf b1,
                       ProbDev* prob, int64_t off_u, int64_t off_d, int K, int nvar, int64_t ncell,
                       const PackOp& op, hipStream_t s) {
    auto* f = prec == P_F64 ? pack_launch<double, double>
              : prec == P_F32 ? pack_launch<float, float>
              : prec == P_ACC64 ? pack_launch<double, float> : pack_launch<ffs, float>;
    f(src, dst, b0, b1, prob, off_u, off_d, K, nvar, ncell, op, s);
    return hipGetLastError();
}

}  // namespace hweno
