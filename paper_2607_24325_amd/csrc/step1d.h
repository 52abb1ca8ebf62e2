// One whole SSP-RK3 step of 1D problems in one kernel (Sec. 2.1 Steps 1-4,
// all three stages), with the step length and the step's end.
//
// A stage reads two cells to either side of a cell, so three stages need six:
// a wave loads 64 * CPT consecutive cells (CPT per lane) with six halo cells
// at each end, carries its cells through the three stages in registers and
// writes the 64 * CPT - 12 inner ones.  Neighbours come from the lane's own
// registers or from the adjacent lane by a DPP shift; there is no barrier and
// no exchange between waves.  The new state goes to the problem's other state
// set (ProbDev::cur), because neighbouring waves still read the old one.
// Every halo cell repeats the arithmetic of its own wave on the same values,
// so both sides of a wave boundary form the same flux bits.
//
// What bounds it and why this split.  A kernel per stage moves 6 state sets,
// three saved sets and two average sets through HBM per step (300 bytes a
// cell in F32_ACC64, 408 in FP64); this one reads and writes the state once
// (72 and 96 bytes): 4.2 million cells of F32_ACC64 take 150 us a step instead
// of 354, and are then bound by vector instructions (all issue slots taken).  On
// small problems the launches were the time (a step was five of them and is
// one: 4000 cells in F64, 10 us instead of 24, of which 1.1 are the loads, 3.8
// the stages and 3.8 the atomics that end the step).  CPT trades halo work (12
// of 64 or 128 cells) against the length of a lane's serial chain and its
// registers (148 and 206 in F64, 96 and 128 in F32_ACC64); see step1d_cells.
#pragma once

#include "stage1d.h"

namespace hweno {

// What the three stages of a wave's cells need besides the cells.
template <class T, class TA> struct Wave1D {
    int g0, nx, bcx;   // first cell of the wave (halo included), cells, boundary
    bool refill;       // ghost cells in the wave that are not periodic images
    T dx, inv_dx, ha, dtt;   // ha: half the Lax-Friedrichs speed
    TA inv_dx_a, dta;
};
template <class T, class TA>
__device__ __forceinline__ Wave1D<T, TA> wave1d(const ProbDev& P, double dt, int g0, int n) {
    Wave1D<T, TA> w;
    w.g0 = g0;
    w.nx = P.nx;
    w.bcx = P.bc_x;
    // images of a periodic domain evolve as the cells they repeat; other
    // ghost cells are set anew from the interior in every stage
    w.refill = P.bc_x != BC_PERIODIC && (g0 < 0 || g0 + n > P.nx);
    w.dx = (T)P.dx;
    w.inv_dx = (T)P.inv_dx;
    w.ha = (T)0.5 * (T)as_double(P.ax_bits);
    w.dtt = (T)dt;
    w.inv_dx_a = (TA)P.inv_dx;
    w.dta = (TA)dt;
    return w;
}

// LDS written by some lanes of a wave is read by others.
__device__ __forceinline__ void wave_lds_sync() {
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    __builtin_amdgcn_wave_barrier();
}

// Takes a wave's cells (u, v), CPT per lane, from U^n to U^(n+1).  gu, gv: LDS
// of the wave alone, for the ghost refill.
template <int P, int K, int FLUX, bool CH, int CPT, class TU, class TD, class T, class TA>
__device__ __forceinline__ void advance1d(TU (&u)[K][CPT], TD (&v)[K][CPT], const Wave1D<T, TA>& w,
                                          const Scheme& sch, TU (*gu)[64 * CPT],
                                          TD (*gv)[64 * CPT]) {
    constexpr int N = 64 * CPT;
    const int lane = threadIdx.x & 63;
    const int squared = sch.weights == W_BETA2;   // W_PAPER prints beta + eps in 1D
    const Flux<T, FLUX, K, 0> F(sch);
    const T g0inv = (T)(1.0 / sch.gam[0]);
    const T dx = w.dx, inv_dx = w.inv_dx, ha = w.ha, dtt = w.dtt;
    const TA inv_dx_a = w.inv_dx_a, dta = w.dta;
    const int g0 = w.g0, nx = w.nx, bcx = w.bcx;
    const bool refill = w.refill;
    TU un[K][CPT];
    TD hn[K][CPT] = {};
#pragma unroll
    for (int c = 0; c < K; ++c)
#pragma unroll
        for (int j = 0; j < CPT; ++j) un[c][j] = u[c][j];
#pragma unroll 1
    for (int s = 0; s < 3; ++s) {
        // faces of the lane's cells: right (u, u_x) of the one before,
        // left of the first cell for the lane to the left.  What a
        // kernel per stage would pass through memory is handed on
        // rounded, so that every place in a wave rounds alike.
        T L0u[K], L0v[K], Ru[K], Rv[K];
        T o2[K][CPT];               // u(x+1/2) - u(x-1/2)
        T f[K][CPT], h[K][CPT];     // fluxes at the right faces
#pragma unroll
        for (int j = 0; j < CPT; ++j) {
            T dm[K], dp[K], vm[K], vp[K], Uc[K], E[K], O[K], De[K], Do[K];
#pragma unroll
            for (int c = 0; c < K; ++c) {
                const TU uc = u[c][j];
                const TU ul = j > 0 ? u[c][j > 0 ? j - 1 : 0] : from_left(u[c][CPT - 1]);
                const TU ur = j < CPT - 1 ? u[c][j < CPT - 1 ? j + 1 : 0] : from_right(u[c][0]);
                const TD vl = j > 0 ? v[c][j > 0 ? j - 1 : 0] : from_left(v[c][CPT - 1]);
                const TD vr = j < CPT - 1 ? v[c][j < CPT - 1 ? j + 1 : 0] : from_right(v[c][0]);
                Uc[c] = (T)uc;
                dm[c] = (T)(ul - uc);
                dp[c] = (T)(ur - uc);
                vm[c] = (T)vl;
                vp[c] = (T)vr;
            }
            recon1d_cell<T, K, CH>(Uc, dm, dp, vm, vp, dx, sch, squared, g0inv, E, O, De, Do);
            T Lu[K], Lv[K];
#pragma unroll
            for (int c = 0; c < K; ++c) {
                Lu[c] = Uc[c] + (E[c] - O[c]);
                Lv[c] = (De[c] - Do[c]) * inv_dx;
                o2[c][j] = (T)2 * O[c];
                handed_on(Lu[c]);
                handed_on(Lv[c]);
                handed_on(o2[c][j]);
            }
            if (j == 0) {
#pragma unroll
                for (int c = 0; c < K; ++c) {
                    L0u[c] = Lu[c];
                    L0v[c] = Lv[c];
                }
            } else {
                T ff_[K], hh_[K];
                lf_interface<P, T, FLUX, K>(F, Ru, Rv, Lu, Lv, ha, ff_, hh_);
#pragma unroll
                for (int c = 0; c < K; ++c) {
                    handed_on(ff_[c]);
                    handed_on(hh_[c]);
                    f[c][j - 1] = ff_[c];
                    h[c][j - 1] = hh_[c];
                }
            }
#pragma unroll
            for (int c = 0; c < K; ++c) {
                Ru[c] = Uc[c] + (E[c] + O[c]);
                Rv[c] = (De[c] + Do[c]) * inv_dx;
                handed_on(Ru[c]);
                handed_on(Rv[c]);
            }
        }
        {
            T Lu[K], Lv[K], ff_[K], hh_[K];
#pragma unroll
            for (int c = 0; c < K; ++c) {
                Lu[c] = from_right(L0u[c]);
                Lv[c] = from_right(L0v[c]);
            }
            lf_interface<P, T, FLUX, K>(F, Ru, Rv, Lu, Lv, ha, ff_, hh_);
#pragma unroll
            for (int c = 0; c < K; ++c) {
                handed_on(ff_[c]);
                handed_on(hh_[c]);
                f[c][CPT - 1] = ff_[c];
                h[c][CPT - 1] = hh_[c];
            }
        }
        // residual and RK combination
#pragma unroll
        for (int c = 0; c < K; ++c) {
            T fl = from_left(f[c][CPT - 1]), hl = from_left(h[c][CPT - 1]);
#pragma unroll
            for (int j = 0; j < CPT; ++j) {
                const TA nLu = ((TA)f[c][j] - (TA)fl) * inv_dx_a;
                const T nLv = (h[c][j] - hl) * inv_dx;
                fl = f[c][j];
                hl = h[c][j];
                const TA ucur = (TA)u[c][j], un0 = (TA)un[c][j];
                const T hn0 = (T)hn[c][j];
                if (s == 0) {
                    hn[c][j] = (TD)(o2[c][j] * inv_dx);
                    u[c][j] = (TU)rk1d_u<P, K, TA>(1, ucur, un0, nLu, dta);
                    v[c][j] = (TD)rk1d_v<T>(1, o2[c][j], inv_dx, hn0, nLv, dtt);
                } else if (s == 1) {
                    u[c][j] = (TU)rk1d_u<P, K, TA>(2, ucur, un0, nLu, dta);
                    v[c][j] = (TD)rk1d_v<T>(2, o2[c][j], inv_dx, hn0, nLv, dtt);
                } else {
                    u[c][j] = (TU)rk1d_u<P, K, TA>(3, ucur, un0, nLu, dta);
                    v[c][j] = (TD)rk1d_v<T>(3, o2[c][j], inv_dx, hn0, nLv, dtt);
                }
            }
        }
        if (refill && s < 2) {
#pragma unroll
            for (int j = 0; j < CPT; ++j)
#pragma unroll
                for (int c = 0; c < K; ++c) {
                    gu[c][lane * CPT + j] = u[c][j];
                    gv[c][lane * CPT + j] = v[c][j];
                }
            wave_lds_sync();
#pragma unroll
            for (int j = 0; j < CPT; ++j) {
                const int g = g0 + lane * CPT + j;
                // the image of a cell up to six beyond the domain is
                // in the wave; the clamp covers lanes without a use
                const int k = min(max(bc_map(g, nx, bcx) - g0, 0), N - 1);
                const bool mir = FLUX == F_EULER && wall_mirrored(g, nx, bcx);
                if (g < 0 || g >= nx) {
#pragma unroll
                    for (int c = 0; c < K; ++c) {
                        u[c][j] = neg_if(gu[c][k], mir && c == 1);
                        v[c][j] = neg_if(gv[c][k], mir && c != 1);
                    }
                }
            }
            wave_lds_sync();
        }
    }
}

// Waves per SIMD the register allocation must allow.  Two cells per lane in
// single precision, component-wise, take 132 registers by themselves; at 128
// (16 bytes of scratch) a fourth wave fits: 4 million cells of F32_ACC64 150
// instead of 168 us a step.  Elsewhere the compiler's own choice is as good
// or a further wave would spill (FP64, one cell: 20-40% slower).
template <int P, bool CH, int CPT> constexpr int step1d_min_waves() {
    return CPT == 2 && P != P_F64 && !CH ? 4 : 1;
}

template <int P, int K, int FLUX, bool CH, int CPT>
__global__ void __launch_bounds__(64, (step1d_min_waves<P, CH, CPT>())) step1d_kernel(Step1Args a) {
    using TU = typename PrecT<P>::TU;
    using TD = typename PrecT<P>::TD;
    using T = typename PrecT<P>::T;
    using TA = typename PrecT<P>::TA;
    constexpr int N = 64 * CPT;          // cells of a wave
    constexpr int OUT = N - STEP1D_HALO; // of which it writes
    __shared__ TU gu[K][N];              // ghost refill of the tiles at a boundary
    __shared__ TD gv[K][N];

    const int lane = threadIdx.x;
    const Scheme& sch = a.sch;

    for (int tix = blockIdx.x; tix < a.ntiles; tix += gridDim.x) {
        const Tile1D tile = a.tiles[tix];
        ProbDev& P_ = a.probs[tile.prob];
        const int slot = (tile.c0 / OUT) & (SLOTS - 1);
        const StepChoice step = choose_step(P_, a.ctl, a.flags);
        if (step.act) {
            const int nx = P_.nx, bcx = P_.bc_x, cur = P_.cur;
            const int64_t off_u = P_.off_u, off_d = P_.off_d;
            const TU* Iu = (const TU*)(cur ? a.s[1].u : a.s[0].u) + off_u;
            const TD* Iv = (const TD*)(cur ? a.s[1].d : a.s[0].d) + off_d;
            TU* Ou = (TU*)(cur ? a.s[0].u : a.s[1].u) + off_u;
            TD* Ov = (TD*)(cur ? a.s[0].d : a.s[1].d) + off_d;
            const int g0 = tile.c0 - 6;              // first cell of the wave
            const Wave1D<T, TA> w = wave1d<T, TA>(P_, step.dt, g0, N);
            TU u[K][CPT];
            TD v[K][CPT];
#pragma unroll
            for (int j = 0; j < CPT; ++j) {
                const int g = g0 + lane * CPT + j;
                const int src = bc_map(g, nx, bcx);
                const bool mir = FLUX == F_EULER && wall_mirrored(g, nx, bcx);
#pragma unroll
                for (int c = 0; c < K; ++c) {
                    u[c][j] = neg_if(Iu[(int64_t)c * nx + src], mir && c == 1);
                    v[c][j] = neg_if(Iv[(int64_t)c * nx + src], mir && c != 1);
                }
            }
            advance1d<P, K, FLUX, CH, CPT>(u, v, w, sch, gu, gv);
            // the new state, its largest speed and first non-admissible cell
            double mx = 0.0;
            long long bad = LLONG_MAX;
#pragma unroll
            for (int j = 0; j < CPT; ++j) {
                const int k = lane * CPT + j, g = g0 + k;
                if (k >= 6 && k < 6 + OUT && g < nx) {
                    double uw[K];
#pragma unroll
                    for (int c = 0; c < K; ++c) {
                        Ou[(int64_t)c * nx + g] = u[c][j];
                        Ov[(int64_t)c * nx + g] = v[c][j];
                        uw[c] = (double)u[c][j];
                    }
                    double sx, sy;
                    if (wave_speed<FLUX, 1, K>(uw, sch, sx, sy)) mx = fmax(mx, sx);
                    else bad = g < bad ? g : bad;
                }
            }
            mx = wave_max_d(mx);
            if (__any(bad != LLONG_MAX)) bad = wave_min_ll(bad);
            if (lane == 0) publish_speeds(P_, tile.prob, a.ctl, slot, mx, 0.0, bad);
        }
        end_tile(P_, tile.prob, slot, a.ctl, a.flags);
    }
}

template <int P, int K, int FLUX, bool CH>
void step1d_launch_cells(int cells, const Step1Args& a, int grid, hipStream_t s) {
    if (cells == 1) step1d_kernel<P, K, FLUX, CH, 1><<<grid, 64, 0, s>>>(a);
    else step1d_kernel<P, K, FLUX, CH, 2><<<grid, 64, 0, s>>>(a);
}

template <int P>
hipError_t step1d_launch_prec(int flux, int cells, const Step1Args& a, int grid, hipStream_t s) {
    if (flux == F_ADV) step1d_launch_cells<P, 1, F_ADV, false>(cells, a, grid, s);
    else if (flux == F_BURGERS) step1d_launch_cells<P, 1, F_BURGERS, false>(cells, a, grid, s);
    else if (a.sch.charwise) step1d_launch_cells<P, 3, F_EULER, true>(cells, a, grid, s);
    else step1d_launch_cells<P, 3, F_EULER, false>(cells, a, grid, s);
    return hipGetLastError();
}

}  // namespace hweno
