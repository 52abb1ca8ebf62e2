// Fused 1D HWENO stage kernel: reconstruction (Sec. 2.1 Steps 1-3,
// Appendix A; for the Euler equations optionally in local characteristic
// variables, CH), interface values, global Lax-Friedrichs fluxes for f and h,
// the residual of eq. semi-discrete-scheme and the SSP-RK3 stage with the
// modified derivative (Sec. 2.1 Step 4).
//
// A workgroup of 256 threads owns 254 consecutive output cells of one
// problem: it stages the 258 averages and derivative means it needs in LDS
// (coalesced, ghost cells through the boundary index map), reconstructs 256
// cells (one per thread, every component), computes the 255 interface
// fluxes once each, and updates the 254 interior cells.  Right-hand sides and
// the option that reduces the speeds of every stage take this path; other steps
// take all three stages at once (step1d.h).
#pragma once

#include "device_common.h"

namespace hweno {

// RK combination of a cell average u and of its derivative with the negated
// residuals nLu, nLv of the input state: stage s = 1, 2, 3.  un, hn: average
// and modified derivative of U^n; o2: the polynomial's difference over the
// cell, o2 * inv_dx the modified derivative of the input.
// Of a combination's two products the first is fused into the sum, but for
// the averages of systems in F64 and F32 the second.
template <int P, int K, class TA>
__device__ __forceinline__ TA rk1d_u(int s, TA u, TA un, TA nLu, TA dt) {
    const TA t = fused(-dt, nLu, u);
    if (s == 1) return t;
    const TA a = s == 2 ? (TA)0.75 : (TA)(1.0 / 3.0), b = s == 2 ? (TA)0.25 : (TA)(2.0 / 3.0);
    return K > 1 && (P == P_F64 || P == P_F32) ? fused(b, t, a * un) : fused(a, un, b * t);
}
template <class T> __device__ __forceinline__ T rk1d_v(int s, T o2, T inv_dx, T hn, T nLv, T dt) {
    if (s == 1) return fused(-dt, nLv, o2 * inv_dx);
    const T t = fused(inv_dx, o2, -(dt * nLv));
    return fused(s == 2 ? (T)0.75 : (T)(1.0 / 3.0), hn, (s == 2 ? (T)0.25 : (T)(2.0 / 3.0)) * t);
}

// HWENO polynomial of one field (Sec. 2.1 Steps 1-3).  The differences of the
// neighbours' averages from the cell's (dm, dp) and the sum and difference
// (right less left) of dx times their derivative means (sv, dv) give the
// Appendix A quartic (centre average subtracted), the two linear polynomials,
// the weights, and the combined polynomial's even and odd parts at the faces
// (E, O) and of its derivative (De, Do).
template <int K, class T>
__device__ __forceinline__ void recon1d_field(T dm, T dp, T sv, T dv, const Scheme& sch,
                                              int squared, T g0inv, T& E, T& O, T& De, T& Do) {
    T c0v[5];
    const T sm = dm + dp;
    c0v[0] = fused((T)(9.0 / 320.0), dv, (T)(-47.0 / 480.0) * sm);
    c0v[1] = fused((T)(13.0 / 16.0), dp - dm, (T)(-5.0 / 16.0) * sv);
    c0v[2] = K > 1 ? fused((T)(5.0 / 4.0), sm, (T)(-3.0 / 8.0) * dv)
                   : fused((T)(-3.0 / 8.0), dv, (T)(5.0 / 4.0) * sm);
    c0v[3] = fused((T)0.25, sv, (T)0.25 * (dm - dp));
    c0v[4] = fused((T)0.25, dv, (T)-0.5 * sm);
    T beta[3];
    beta[0] = sch.smoothness == BETA_CLASSICAL
                  ? beta_classical_1d(c0v)
                  : c0v[1] * c0v[1] + (T)4 * c0v[2] * c0v[2] + (T)36 * c0v[3] * c0v[3] +
                        (T)576 * c0v[4] * c0v[4];
    beta[1] = dm * dm;
    beta[2] = dp * dp;
    T w[3];
    nonlinear_weights<T, 2>(beta, sch, squared, w);
    const T a0 = w[0] * g0inv;
    const T b1 = w[1] - a0 * (T)sch.gam[1], b2 = w[2] - a0 * (T)sch.gam[2];
    T C[5];
#pragma unroll
    for (int l = 0; l < 5; ++l) C[l] = a0 * c0v[l];
    C[1] += b2 * dp - b1 * dm;   // slopes of p1 (-dm) and p2 (dp)
    E = C[0] + (T)0.25 * C[2] + (T)0.0625 * C[4];
    O = (T)0.5 * C[1] + (T)0.125 * C[3];
    De = C[1] + (T)0.75 * C[3];
    Do = C[2] + (T)0.5 * C[4];
}

// All components of one cell with average Uc (vm, vp: the neighbours'
// derivative means): each by itself, or (CH) in the
// local characteristic variables of the cell's own average.  The
// reconstruction is linear in the stencil except for the weights, so the
// differences project directly and the face values map back with R.
template <class T, int K, bool CH>
__device__ __forceinline__ void recon1d_cell(const T* Uc, const T* dm, const T* dp, const T* vm,
                                             const T* vp, T dx, const Scheme& sch, int squared,
                                             T g0inv, T* E, T* O, T* De, T* Do) {
    if constexpr (CH) {
        const Eigen<T> ev(Uc, (T)(sch.gas_gamma - 1.0));
        T dvm[K], dvp[K], wm[K], wp[K], wvm[K], wvp[K], e[K], o[K], de[K], dd[K];
#pragma unroll
        for (int c = 0; c < K; ++c) {
            dvm[c] = dx * vm[c];
            dvp[c] = dx * vp[c];
        }
        ev.left(dm, wm);
        ev.left(dp, wp);
        ev.left(dvm, wvm);
        ev.left(dvp, wvp);
#pragma unroll
        for (int k = 0; k < K; ++k)
            recon1d_field<K, T>(wm[k], wp[k], wvm[k] + wvp[k], wvp[k] - wvm[k], sch, squared, g0inv,
                             e[k], o[k], de[k], dd[k]);
        ev.right(e, E);
        ev.right(o, O);
        ev.right(de, De);
        ev.right(dd, Do);
    } else {
#pragma unroll
        for (int c = 0; c < K; ++c) {
            const T dvp = dx * vp[c];
            recon1d_field<K, T>(dm[c], dp[c], fused(dx, vm[c], dvp), fused(-dx, vm[c], dvp), sch,
                             squared, g0inv, E[c], O[c], De[c], Do[c]);
        }
    }
}

// A value that is handed on as rounded: the compiler may not contract the
// operation that made it with those that use it.  No instruction.
__device__ __forceinline__ void handed_on(float& x) { asm("" : "+v"(x)); }
__device__ __forceinline__ void handed_on(double& x) { asm("" : "+v"(x)); }

// Lax-Friedrichs fluxes f-hat, h-hat at one interface (ha: half the speed).
// Of the two sides' products that are added, one is rounded by itself and the
// other fused into the sum: the left one is rounded for the scalar laws in
// F32_KAHAN, the right one otherwise.
template <int P, class T, int FLUX, int K>
__device__ __forceinline__ void lf_interface(const Flux<T, FLUX, K, 0>& F, const T* UL, const T* VL,
                                             const T* UR, const T* VR, T ha, T* f, T* h) {
    T fL[K], hL[K], fR[K], hR[K];
    F.side(UL, VL, nullptr, fL, hL, nullptr);
    F.side(UR, VR, nullptr, fR, hR, nullptr);
#pragma unroll
    for (int c = 0; c < K; ++c) {
        handed_on(P == P_KAHAN && K == 1 ? fL[c] : fR[c]);
        handed_on(P == P_KAHAN && K == 1 ? hL[c] : hR[c]);
        f[c] = (T)0.5 * (fL[c] + fR[c]) - ha * (UR[c] - UL[c]);
        h[c] = (T)0.5 * (hL[c] + hR[c]) - ha * (VR[c] - VL[c]);
    }
}

// Workgroups per CU the register allocation must allow.  With FP32 faces
// the staging in LDS (21.6 KB per workgroup) admits seven; six fit the
// registers of stages 1-3 (stage 3, with the FP64 wave-speed reduction,
// only because it loads its RK inputs late, see stage1d_late_rk); the
// right-hand side and the characteristic projections need more.  With FP64
// faces LDS (37 KB) admits four and the allocation is left to the compiler.
template <int P, int mode, bool CH> constexpr int stage1d_min_blocks() {
    return P == P_F64 ? 1
                      : CH ? (mode == MODE_S3 ? 4 : 5)
                           : (mode == MODE_RHS ? 5 : 6);
}

// Stage 3 of the Euler system in single precision (component-wise) loads
// U^n and the saved derivatives after the reconstruction instead of before
// it: the nine registers they would hold through it are what separates its
// 95 VGPRs (five workgroups per CU) from 80 (six), and the extra workgroup
// hides more latency than the late loads expose.
template <int P, int K, int mode, bool CH> constexpr bool stage1d_late_rk() {
    return mode == MODE_S3 && P != P_F64 && !CH && K > 1;
}

// Group of a tile among its problem's tiles.
__device__ __forceinline__ int c0_slot(int c0) { return (c0 / TILE1D_OUT) & (SLOTS - 1); }

template <int P, int K, int FLUX, int mode, bool CH>
__global__ void __launch_bounds__(256, (stage1d_min_blocks<P, mode, CH>())) stage1d_kernel(StageArgs a) {
    using TU = typename PrecT<P>::TU;
    using TD = typename PrecT<P>::TD;
    using T = typename PrecT<P>::T;
    using TA = typename PrecT<P>::TA;
    constexpr int NL = TILE1D_OUT + 4;   // staged cells
    __shared__ TU su[K][NL];
    __shared__ TD sv[K][NL];
    __shared__ T sR[2 * K][256];         // (u, u_x) at x_{i+1/2} from cell i
    __shared__ T sL[2 * K][256];         // (u, u_x) at x_{i-1/2} from cell i
    // (f-hat, h-hat) at the right interface of cell t: written over sR, whose
    // entry t only thread t reads (right before it writes the flux there)
    T (&sF)[2 * K][256] = sR;
    __shared__ double s_mx[4];           // stage 3: per-wave maxima of the wave speeds
    __shared__ long long s_bad[4];

    const int tid = threadIdx.x;
    const Scheme& sch = a.sch;
    const int squared = sch.weights == W_BETA2;   // W_PAPER prints beta + eps in 1D
    const Flux<T, FLUX, K, 0> F(sch);
    const Tile1D* tiles = (const Tile1D*)a.tiles + a.tile_offset;
    const T g0inv = (T)(1.0 / sch.gam[0]);

    for (int tix = blockIdx.x; tix < a.ntiles; tix += gridDim.x) {
        const Tile1D tile = tiles[tix];
        ProbDev& P_ = a.probs[tile.prob];
        const int slot = c0_slot(tile.c0);
        StepChoice step{};
        if (mode != MODE_RHS) {
            step = stage_step(P_, a.ctl, a.flags, mode);
            if (!step.act) {
                if (mode == MODE_S3 && tid < 64)
                    publish_and_end(&P_, tile.prob, slot, a.ctl, a.flags, 0, 0.0, 0.0, LLONG_MAX);
                continue;
            }
        }
        const int nx = P_.nx, bcx = P_.bc_x;
        const T dx = (T)P_.dx, inv_dx = (T)P_.inv_dx;
        const TA inv_dx_a = (TA)P_.inv_dx;
        const T alpha = (T)as_double(P_.ax_bits);
        const double dt = step.dt;
        const int c0 = tile.c0;
        // problem-table fields are copied before any store: read after one,
        // they would be reloaded (possible aliasing) and waited for
        const int64_t off_u = P_.off_u, off_d = P_.off_d;
        const StateBuf in = mode == MODE_RHS && P_.cur ? a.in1 : a.in;

        for (int k = tid; k < NL; k += 256) {
            const int src = bc_map(c0 - 2 + k, nx, bcx);
            const bool mir = FLUX == F_EULER && wall_mirrored(c0 - 2 + k, nx, bcx);
#pragma unroll
            for (int c = 0; c < K; ++c) {
                // behind a wall: momentum odd, other averages even, and the
                // derivative means of the opposite parity
                su[c][k] = neg_if(((const TU*)in.u)[off_u + (int64_t)c * nx + src], mir && c == 1);
                sv[c][k] = neg_if(((const TD*)in.d)[off_d + (int64_t)c * nx + src], mir && c != 1);
            }
        }
        // stages 2 and 3: U^n and the saved derivatives of the output cell
        // (lanes without output read element 0), loaded now so that they
        // arrive while the cell is reconstructed and the fluxes are formed,
        // or after the reconstruction (stage1d_late_rk)
        const int gi = c0 - 1 + tid;
        const bool emit = tid >= 1 && tid <= TILE1D_OUT && gi < nx;
        constexpr bool LATE_RK = stage1d_late_rk<P, K, mode, CH>();
        TA unr[K];
        T hnr[K];
        auto load_rk = [&]() {
            const int gl = emit ? gi : 0;
#pragma unroll
            for (int c = 0; c < K; ++c) {
                unr[c] = (TA)((const TU*)a.un)[off_u + (int64_t)c * nx + gl];
                hnr[c] = (T)((const TD*)a.h)[off_d + (int64_t)c * nx + gl];
            }
        };
        if constexpr ((mode == MODE_S2 || mode == MODE_S3) && !LATE_RK) load_rk();
        __syncthreads();

        // ---- reconstruct local cell tid (global c0 - 1 + tid) ---------------
        T dm[K], dp[K], vm[K], vp[K], Uc[K], E[K], O[K], De[K], Do[K];
#pragma unroll
        for (int c = 0; c < K; ++c) {
            const TU uc = su[c][tid + 1];
            Uc[c] = (T)uc;
            dm[c] = (T)(su[c][tid] - uc);        // u_{i-1} - u_i
            dp[c] = (T)(su[c][tid + 2] - uc);    // u_{i+1} - u_i
            vm[c] = (T)sv[c][tid];
            vp[c] = (T)sv[c][tid + 2];
        }
        recon1d_cell<T, K, CH>(Uc, dm, dp, vm, vp, dx, sch, squared, g0inv, E, O, De, Do);
        T o2[K];   // u(x+1/2) - u(x-1/2)
#pragma unroll
        for (int c = 0; c < K; ++c) {
            const T ucT = (T)su[c][tid + 1];
            sR[c][tid] = ucT + (E[c] + O[c]);
            sL[c][tid] = ucT + (E[c] - O[c]);
            sR[K + c][tid] = (De[c] + Do[c]) * inv_dx;
            sL[K + c][tid] = (De[c] - Do[c]) * inv_dx;
            o2[c] = (T)2 * O[c];
        }
        if constexpr (LATE_RK) load_rk();
        __syncthreads();

        // ---- flux at the interface between local cells tid and tid+1 -------
        if (tid < 255) {
            T UL[K], VL[K], UR[K], VR[K], f[K], h[K];
#pragma unroll
            for (int c = 0; c < K; ++c) {
                UL[c] = sR[c][tid]; VL[c] = sR[K + c][tid];
                UR[c] = sL[c][tid + 1]; VR[c] = sL[K + c][tid + 1];
            }
            lf_interface<P, T, FLUX, K>(F, UL, VL, UR, VR, (T)0.5 * alpha, f, h);
#pragma unroll
            for (int c = 0; c < K; ++c) {
                sF[c][tid] = f[c];
                sF[K + c][tid] = h[c];
            }
        }
        __syncthreads();

        // ---- residual and RK stage of local cell tid -----------------------
        double unew[K];
        if (emit) {
#pragma unroll
            for (int c = 0; c < K; ++c) {
                const TA nLu = ((TA)sF[c][tid] - (TA)sF[c][tid - 1]) * inv_dx_a;
                const T nLv = (sF[K + c][tid] - sF[K + c][tid - 1]) * inv_dx;
                const TA ucur = (TA)su[c][tid + 1];
                const int64_t ou = off_u + (int64_t)c * nx + gi;
                const int64_t od = off_d + (int64_t)c * nx + gi;
                if (mode == MODE_RHS) {
                    const int64_t ob = (int64_t)c * nx + gi;
                    a.L_out[ob] = (double)(-nLu);
                    a.L_out[(int64_t)K * nx + ob] = (double)(-nLv);
                    a.Uh_out[ob] = (double)ucur;
                    a.Uh_out[(int64_t)K * nx + ob] = (double)(o2[c] * inv_dx);
                } else {
                    if (mode == MODE_S1) {
                        unr[c] = 0;
                        hnr[c] = 0;
                        ((TD*)a.h)[od] = (TD)(o2[c] * inv_dx);
                    }
                    const TU nu = (TU)rk1d_u<P, K, TA>(mode, ucur, unr[c], nLu, (TA)dt);
                    ((TU*)a.out.u)[ou] = nu;
                    ((TD*)a.out.d)[od] = (TD)rk1d_v<T>(mode, o2[c], inv_dx, hnr[c], nLv, (T)dt);
                    if (mode == MODE_S3) unew[c] = (double)nu;
                }
            }
        }
        if (mode == MODE_S3) {
            // largest x wave speed of the state being written (the 1D time
            // step uses no other), for the next step: reduced over the wave
            // here and over the workgroup below; the first non-admissible
            // cell is reduced only where there is one
            double mx = 0.0;
            long long bad = LLONG_MAX;
            if (emit) {
                double sx, sy;
                if (wave_speed<FLUX, 1, K>(unew, sch, sx, sy)) mx = sx;
                else bad = gi;
            }
            mx = wave_max_d(mx);
            if (__any(bad != LLONG_MAX)) bad = wave_min_ll(bad);
            if ((tid & 63) == 0) {
                s_mx[tid >> 6] = mx;
                s_bad[tid >> 6] = bad;
            }
        }
        __syncthreads();   // LDS reuse by the next tile
        if (mode == MODE_S3 && tid < 64) {
            double mx = s_mx[0];
            long long bad = s_bad[0];
#pragma unroll
            for (int w = 1; w < 4; ++w) {
                mx = fmax(mx, s_mx[w]);
                bad = s_bad[w] < bad ? s_bad[w] : bad;
            }
            publish_and_end(&P_, tile.prob, slot, a.ctl, a.flags, 1, mx, 0.0, bad);
        }
    }
}

}  // namespace hweno
