// 2D Euler stage kernel with the HWENO reconstruction and derivative
// modification in local characteristic variables (remark closing Sec. 2.2):
// each cell's stencil is projected with the eigenvectors of the flux
// Jacobian at the cell's own average, once with those of F (x) and once with
// those of G (y); every characteristic field is reconstructed as a scalar
// (Sec. 2.2 Steps 1-3, Appendix A), the x-edge values and v-hat come from the
// x-projected polynomials and the y-edge values and w-hat from the
// y-projected ones, and are mapped back to conserved variables with R.
// Fluxes, residual and RK stage are those of the component-wise kernel.
//
// Work decomposition as in stage2d_kernel (64-column strip, rows marched
// upwards, wave k = characteristic field k in R, face k in F and component k in
// the loads and in S, lane = column), with one change: a projection mixes all
// four components of every stencil entry, so what the stencils of a row are
// made of lives in LDS, where every wave reads it: the averages' differences to
// the right and upper neighbours in working precision (each formed once from
// the wide averages, a corner being a sum of two) and the derivative averages.
// Per row r:
//   top  each wave writes its component of row r+1's differences and of row
//        r+2's derivative averages (loaded one row earlier);
//   R    wave k projects the stencil of its lane's cell with row k of L_x and
//        of L_y, reconstructs both fields and writes the face values as
//        characteristic differences from the cell average to LDS;
//   F    wave k forms the conserved values at the points of face k of its
//        lane's cell from the four fields and sums that side of the
//        Lax-Friedrichs flux; two waves also map the hats back;
//   S    residual and RK stage of row r-1, as in the component-wise kernel.
// Bound by vector instructions.  A face belongs to one cell, so an edge point
// needs one set of eigenvectors, which R has formed already, instead of two
// formed again for each point, the row of L is one expression for all fields
// (no selection by the wave's field), and R is applied in factored form: 25.0
// million instructions a stage of 768 x 512 cells in F32_ACC64 instead of 35.2,
// in 155 instead of 220 registers and 43 instead of 55 KB of LDS, so that three
// workgroups instead of two share a CU: 56 us instead of 71.
#pragma once

#include "stage2d.h"

namespace hweno {

// Eigenvectors of the x and y flux Jacobians at a cell's average: columns of R
// (rows of L = R^-1), in the order (rho, m_n, m_t, E) with m_n the momentum
// along the direction, belong to v_n - c, v_n, v_n (shear), v_n + c.  The two
// directions differ only in which velocity is v_n.
template <class T> struct Eigen2 {
    T u, v, c, H, hq2, b1, b2, ec;
    __device__ __forceinline__ Eigen2(const T* U, T gm1) {
        const T ir = rcp(U[0]);
        u = U[1] * ir;
        v = U[2] * ir;
        hq2 = (T)0.5 * fused(u, u, v * v);
        const T p = gm1 * fused(-U[0], hq2, U[3]);
        c = sqrt((gm1 + (T)1) * p * ir);
        const T ic = rcp(c);
        H = (U[3] + p) * ir;
        b1 = gm1 * ic * ic;
        b2 = b1 * hq2;
        ec = (T)0.5 * ic;
    }
};
// Row of L of one field, with the field's (wave-uniform) factors:
//   v -+ c:  b2/2 +- vn ec,  -b1 vn/2 -+ ec,  -b1 vt/2,  b1/2
//   v:       1 - b2,          b1 vn,           b1 vt,    -b1
//   shear:   -vt,             0,               1,         0
template <class T> struct LRow {
    T one, b, s, t;   // row = b (b2, -b1 vn, -b1 vt, b1) + one e0 + s (vn ec, -ec, 0, 0) + t (-vt, 0, 1, 0)
    __device__ __forceinline__ LRow(int field)
        : one(field == 1 ? (T)1 : (T)0), b(field == 1 ? (T)-1 : (field == 2 ? (T)0 : (T)0.5)),
          s(field == 0 ? (T)1 : (field == 3 ? (T)-1 : (T)0)), t(field == 2 ? (T)1 : (T)0) {}
    __device__ __forceinline__ void row(const Eigen2<T>& e, T vn, T vt, T* L) const {
        const T sec = s * e.ec, bb = b * e.b1;
        L[0] = fused(b, e.b2, fused(vn, sec, fused(-t, vt, one)));
        L[1] = -fused(bb, vn, sec);
        L[2] = fused(-bb, vt, t);
        L[3] = bb;
    }
};
// x = R w.
template <class T>
__device__ __forceinline__ void from_fields(T vn, T vt, T c, T H, T hq2, const T* w, T* x) {
    const T s = w[0] + w[3], cd = c * (w[3] - w[0]);
    x[0] = s + w[1];
    x[1] = fused(vn, x[0], cd);
    x[2] = fused(vt, x[0], w[2]);
    x[3] = fused(H, s, fused(hq2, w[1], fused(vt, w[2], vn * cd)));
}

// Workgroups per CU: three in single precision (up to 160 registers; 43 KB of
// LDS with two Gauss points, with three of them 55 KB allow two), one in FP64.
template <int P, int Q, int mode>
__global__ void __launch_bounds__(256, (P == P_F64 ? 1 : 3)) stage2d_char_kernel(StageArgs a) {
    constexpr int K = 4;
    using TU = typename PrecT<P>::TU;
    using TD = typename PrecT<P>::TD;
    using T = typename PrecT<P>::T;
    using TA = typename PrecT<P>::TA;
    // characteristic differences at the Gauss points of the four faces, then
    // the faces' sides of the flux, as in stage2d_kernel
    __shared__ T sF[4][Q * 3 * K][64];
    __shared__ T sU[2][K][64], sDx[2][K][64];   // averages; differences to the right
    __shared__ T sDy[4][K][64];                 // differences to the row above
    __shared__ TD sV[4][K][64], sW[4][K][64];   // derivative averages
    __shared__ T sH[2][K][64];                  // hats: characteristic, then conserved
    __shared__ double smx[K], smy[K];           // stage 3, as in stage2d_kernel
    __shared__ long long sbad[K];

    const int lane = threadIdx.x & 63;
    const int c = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const Scheme& sch = a.sch;
    const int squared = sch.weights == W_BETA2 || (sch.weights == W_PAPER);
    const Flux<T, F_EULER, K, 0> FXf(sch);
    const Flux<T, F_EULER, K, 1> FYf(sch);
    const T gm1 = (T)(sch.gas_gamma - 1.0);
    const LRow<T> lrow(c);
    const Tile2D* tiles = (const Tile2D*)a.tiles + a.tile_offset;
    // y-direction component order (rho, m_y, m_x, E) -> storage index
    constexpr int PY[4] = {0, 2, 1, 3};

    for (int tix = blockIdx.x; tix < a.ntiles; tix += gridDim.x) {
        const Tile2D tile = tiles[tix];
        const ProbDev& P_ = a.probs[tile.prob];
        StepChoice step{};
        if (mode != MODE_RHS) {
            step = stage_step(P_, a.ctl, a.flags, mode);
            if (!step.act) {
                if (mode == MODE_S3 && c == 0)
                    publish_and_end(&a.probs[tile.prob], tile.prob, tile.slot, a.ctl, a.flags, 0,
                                    0.0, 0.0, LLONG_MAX);
                continue;
            }
        }
        const int nx = P_.nx, ny = P_.ny, bcx = P_.bc_x, bcy = P_.bc_y;
        const int64_t plane = (int64_t)nx * ny;
        // the residual's factors, as in stage2d_kernel
        const T inv_dx = (T)(P_.inv_dx * (2.0 * WSUM<Q>)), inv_dy = (T)(P_.inv_dy * (2.0 * WSUM<Q>));
        const TA inv_dx_a = (TA)(P_.inv_dx * WSUM<Q>), inv_dy_a = (TA)(P_.inv_dy * WSUM<Q>);
        const T rx = (T)(P_.dx * P_.inv_dy), ry = (T)(P_.dy * P_.inv_dx);
        const T ax = (T)as_double(P_.ax_bits), ay = (T)as_double(P_.ay_bits);
        const double dt = step.dt;
        const int gi = tile.i0 - 2 + lane;
        const int li = bc_map(gi, nx, bcx);
        const bool out_col = lane >= 2 && lane < 62 && gi < nx;
        const int64_t off_u = P_.off_u, off_d = P_.off_d;
        const TU* Uu = (const TU*)a.in.u + off_u + c * plane;
        const TD* Uv = (const TD*)a.in.d + off_d + c * plane;
        const TD* Uw = (const TD*)a.in.d + off_d + (K + c) * plane;
        const TU* Un = (const TU*)a.un + off_u + c * plane;
        TD* Hv = (TD*)a.h + off_d + c * plane;
        TD* Hw = (TD*)a.h + off_d + (K + c) * plane;
        TU* Ou = (TU*)a.out.u + off_u + c * plane;
        TD* Ov = (TD*)a.out.d + off_d + c * plane;
        TD* Ow = (TD*)a.out.d + off_d + (K + c) * plane;

        const bool mx = wall_mirrored(gi, nx, bcx);
        const bool nux = mx && c == 1, nvx = mx && c != 1, nwx = mx && c == 1;
        auto load_row = [&](int j, TU& u, TD& v, TD& w) {
            const uint32_t o = (uint32_t)(bc_map(j, ny, bcy) * nx + li);
            const bool my = wall_mirrored(j, ny, bcy);
            const bool nuy = my && c == 2, nvy = my && c == 2, nwy = my && c != 2;
            u = neg_if(plane_at(Uu, o), nux != nuy);
            v = neg_if(plane_at(Uv, o), nvx != nvy);
            w = neg_if(plane_at(Uw, o), nwx != nwy);
        };
        auto put_derivs = [&](int j, TD v, TD w) {
            sV[j & 3][c][lane] = v;
            sW[j & 3][c][lane] = w;
        };
        // row j's differences from its averages u and those of the row above
        auto put_diffs = [&](int j, TU u, TU above) {
            sU[j & 1][c][lane] = (T)u;
            sDx[j & 1][c][lane] = (T)(from_right(u) - u);
            sDy[j & 3][c][lane] = (T)(above - u);
        };
        const int j0 = tile.j0, jend = tile.j0 + tile.nrows;

        // prologue: what row j0-1's stencils are made of; row j0+1 prefetched
        TU um, u0, up, un_;
        TD vn_, wn_;
        {
            TD v, w;
            load_row(j0 - 2, um, v, w);
            put_derivs(j0 - 2, v, w);
            load_row(j0 - 1, u0, v, w);
            put_derivs(j0 - 1, v, w);
            load_row(j0, up, v, w);
            put_derivs(j0, v, w);
            put_diffs(j0 - 2, um, u0);
            put_diffs(j0 - 1, u0, up);
        }
        load_row(j0 + 1, un_, vn_, wn_);
        __syncthreads();

        T top_prev[3] = {0, 0, 0};
        // previous row's flux sums: x differences and y sums of the
        // cell-average fluxes in the accumulation type, of the derivative
        // fluxes in T
        TA xdu_prev = 0, gyu_prev = 0;
        T xdd_prev[2] = {0, 0}, gyd_prev[2] = {0, 0};
        T hat_prev[2] = {0, 0};
        const int lm = lane > 0 ? lane - 1 : 0, lp = lane < 63 ? lane + 1 : 63;

        for (int r = j0 - 1; r <= jend; ++r) {
            // row r+2's averages arrive: row r+1's differences are known
            const TU u2 = un_;
            put_diffs(r + 1, up, u2);
            put_derivs(r + 2, vn_, wn_);
            load_row(r + 3, un_, vn_, wn_);

            TA unr = 0;
            T hvr = 0, hwr = 0;
            const bool emit = r > j0 && out_col;
            const uint32_t oo = (uint32_t)((r - 1) * nx + gi);
            if (mode == MODE_S2 || mode == MODE_S3) {
                const uint32_t ol = emit ? oo : 0u;
                unr = (TA)plane_at(Un, ol);
                hvr = (T)plane_at(Hv, ol);
                hwr = (T)plane_at(Hw, ol);
            }

            // ---- R: field c of the cell (gi, r), in x and y projections ----
            // the rows beside the segment only lend it a y edge
            const bool inner = r >= j0 && r < jend;
            const int sm = (r - 1) & 3, s0 = r & 3, sp = (r + 1) & 3, sd = r & 1;
            T en, et, ecs, eH, eq;   // the eigenvectors of this wave's face
            T Lx[K], Ly[K];
            {
                T Uc[K];
#pragma unroll
                for (int k = 0; k < K; ++k) Uc[k] = sU[sd][k][lane];
                const Eigen2<T> e(Uc, gm1);
                lrow.row(e, e.u, e.v, Lx);
                lrow.row(e, e.v, e.u, Ly);
                en = c < 2 ? e.u : e.v;
                et = c < 2 ? e.v : e.u;
                ecs = e.c;
                eH = e.H;
                eq = e.hq2;
            }
            // The stencil in field c: projected differences, then the entries.
            // (One direction at a time: its LDS reads are repeated for the
            // other, for 17 registers less.)
            auto stencil = [&](const T* L, T* q) {
                T d[16];
#pragma unroll
                for (int k = 0; k < K; ++k) {
                    const T x[16] = {sDx[sd][k][lm],     sDx[sd][k][lane],
                                     sDy[sm][k][lm],     sDy[sm][k][lane], sDy[sm][k][lp],
                                     sDy[s0][k][lm],     sDy[s0][k][lane], sDy[s0][k][lp],
                                     (T)sV[s0][k][lm],   (T)sV[s0][k][lp],
                                     (T)sV[sm][k][lane], (T)sV[sp][k][lane],
                                     (T)sW[s0][k][lm],   (T)sW[s0][k][lp],
                                     (T)sW[sm][k][lane], (T)sW[sp][k][lane]};
#pragma unroll
                    for (int e = 0; e < 16; ++e) d[e] = k == 0 ? L[k] * x[e] : fused(L[k], x[e], d[e]);
                }
                q[0] = -d[2] - d[0];
                q[1] = -d[3];
                q[2] = d[1] - d[4];
                q[3] = -d[0];
                q[4] = (T)0;
                q[5] = d[1];
                q[6] = d[5] - d[0];
                q[7] = d[6];
                q[8] = d[7] + d[1];
#pragma unroll
                for (int e = 9; e < 17; ++e) q[e] = d[e - 1];
                asm volatile("" ::: "memory");
            };
            // Derivatives in local units (d/dX, d/dY): the back projection and
            // the edge flux are linear in them, and the residual applies 2/dx,
            // 2/dy once.
            auto put = [&](int f, const T (*val)[Q], const T (*dX)[Q], const T (*dY)[Q]) {
#pragma unroll
                for (int mu = 0; mu < Q; ++mu) {
                    sF[f][(mu * 3 + 0) * K + c][lane] = val[f & 1][mu];
                    sF[f][(mu * 3 + 1) * K + c][lane] = dX[f & 1][mu];
                    sF[f][(mu * 3 + 2) * K + c][lane] = dY[f & 1][mu];
                }
            };
            if (inner) {
                T q[17], C[15], vh, wh, val[2][Q], dn[2][Q], dtg[2][Q], half[2];
                stencil(Lx, q);
                reconstruct2d<T>(q, sch, squared, C, vh, wh);
                face_values<T, Q>(C, val, dn, dtg, half);
                put(0, val, dn, dtg);
                put(1, val, dn, dtg);
                sH[0][c][lane] = vh;
            }
            {
                T q[17], C[15], D[15], vh, wh, val[2][Q], dn[2][Q], dtg[2][Q], half[2];
                // storage component k is position PY[k] of the y order
                const T L[K] = {Ly[PY[0]], Ly[PY[1]], Ly[PY[2]], Ly[PY[3]]};
                stencil(L, q);
                reconstruct2d<T>(q, sch, squared, C, vh, wh);
                transpose15(C, D);
                face_values<T, Q>(D, val, dn, dtg, half);
                put(2, val, dtg, dn);
                put(3, val, dtg, dn);
                sH[1][c][lane] = wh;
            }
            __syncthreads();  // A: face values and hats of row r ready

            // ---- F: the faces' sides of the edge fluxes ---------------------
            auto face = [&](auto fi, const auto& F, T al) {
                constexpr int f = decltype(fi)::value, dir = f / 2;
                T U[K], out[3 * K];
                T rel[K];   // the values relative to the cell's average, over the points
#pragma unroll
                for (int k = 0; k < K; ++k) U[k] = sU[sd][k][lane];
                lf_face<Q>(F, al, [&](int mu, int v, T* D) {
                    T w[K], x[K];
#pragma unroll
                    for (int k = 0; k < K; ++k) w[k] = sF[f][(mu * 3 + v) * K + k][lane];
                    from_fields(en, et, ecs, eH, eq, w, x);
#pragma unroll
                    for (int k = 0; k < K; ++k) {
                        const int s = dir ? PY[k] : k;
                        D[s] = v == 0 ? U[s] + x[k] : x[k];
                        if (v == 0) {
                            if (mu == (Q == 3 ? 1 : 0)) rel[s] = Q == 3 ? (T)1.6 * x[k] : x[k];
                            else rel[s] += x[k];
                        }
                    }
                }, out);
                // the dissipation of the averages: the faces' part, to which the
                // edge adds that of the averages' difference
#pragma unroll
                for (int k = 0; k < K; ++k) out[k] = fused(al, rel[k], out[k]);
                if (f == 1 || f == 2) {   // v-hat by a wave of an x face, w-hat of a y face
                    T w[K], x[K];
#pragma unroll
                    for (int k = 0; k < K; ++k) w[k] = sH[dir][k][lane];
                    from_fields(en, et, ecs, eH, eq, w, x);
#pragma unroll
                    for (int k = 0; k < K; ++k) sH[dir][dir ? PY[k] : k][lane] = x[k];
                }
#pragma unroll
                for (int k = 0; k < 3 * K; ++k) sF[f][k][lane] = out[k];
            };
            if (inner || c == (r < j0 ? 3 : 2)) {
                if (c == 0) face(std::integral_constant<int, 0>(), FXf, -ax);
                else if (c == 1) face(std::integral_constant<int, 1>(), FXf, ax);
                else if (c == 2) face(std::integral_constant<int, 2>(), FYf, -ay);
                else face(std::integral_constant<int, 3>(), FYf, ay);
            }
            __syncthreads();  // B: fluxes and hats ready
            // ---- S: residual and RK stage of row r-1 ------------------------
            // The derivative fluxes are differenced in T: the difference of
            // two T values rounded to T is what a wider difference rounds to.
            TA xdu = 0, gyu = 0;
            T xdd[2], gyd[2];
#pragma unroll
            for (int sk = 0; sk < 3; ++sk) {
                T fr = sF[1][sk * K + c][lane] + from_right(sF[0][sk * K + c][lane]);
                T g = top_prev[sk] + sF[2][sk * K + c][lane];
                if (sk == 0) {
                    fr = fused(-ax, (T)(2.0 * WHALF<Q>) * sDx[sd][c][lane], fr);
                    g = fused(-ay, (T)(2.0 * WHALF<Q>) * sDy[sm][c][lane], g);
                }
                const T fl = from_left(fr);
                top_prev[sk] = sF[3][sk * K + c][lane];
                if (sk == 0) {
                    xdu = (TA)fr - (TA)fl;
                    gyu = (TA)g;
                } else {
                    xdd[sk - 1] = fr - fl;
                    gyd[sk - 1] = g;
                }
            }
            if (r > j0) {
                const TA Lu = -(xdu_prev * inv_dx_a + (gyu - gyu_prev) * inv_dy_a);
                // v- and w-fluxes carry the derivatives in local units
                const T Lv = -inv_dx * (xdd_prev[0] + rx * (gyd[0] - gyd_prev[0]));
                const T Lw = -inv_dy * (ry * xdd_prev[1] + (gyd[1] - gyd_prev[1]));
                if (emit) {
                    const TA ucur = (TA)um;   // u-bar of row r-1 in the input set
                    if (mode == MODE_RHS) {
                        const int64_t ob = (int64_t)c * plane + oo;
                        a.L_out[ob] = (double)Lu;
                        a.L_out[K * plane + ob] = (double)Lv;
                        a.L_out[2 * K * plane + ob] = (double)Lw;
                        a.Uh_out[ob] = (double)ucur;
                        a.Uh_out[K * plane + ob] = (double)hat_prev[0];
                        a.Uh_out[2 * K * plane + ob] = (double)hat_prev[1];
                    } else {
                        const TA dta = (TA)dt;
                        const T dtt = (T)dt;
                        if (mode == MODE_S1) {
                            plane_at(Ou, oo) = (TU)(ucur + dta * Lu);
                            plane_at(Ov, oo) = (TD)(hat_prev[0] + dtt * Lv);
                            plane_at(Ow, oo) = (TD)(hat_prev[1] + dtt * Lw);
                            plane_at(Hv, oo) = (TD)hat_prev[0];
                            plane_at(Hw, oo) = (TD)hat_prev[1];
                        } else if (mode == MODE_S2) {
                            plane_at(Ou, oo) = (TU)((TA)0.75 * unr + (TA)0.25 * (ucur + dta * Lu));
                            plane_at(Ov, oo) = (TD)((T)0.75 * hvr + (T)0.25 * (hat_prev[0] + dtt * Lv));
                            plane_at(Ow, oo) = (TD)((T)0.75 * hwr + (T)0.25 * (hat_prev[1] + dtt * Lw));
                        } else {
                            const TA third = (TA)(1.0 / 3.0), two3 = (TA)(2.0 / 3.0);
                            plane_at(Ou, oo) = (TU)(third * unr + two3 * (ucur + dta * Lu));
                            plane_at(Ov, oo) = (TD)((T)(1.0 / 3.0) * hvr +
                                          (T)(2.0 / 3.0) * (hat_prev[0] + dtt * Lv));
                            plane_at(Ow, oo) = (TD)((T)(1.0 / 3.0) * hwr +
                                          (T)(2.0 / 3.0) * (hat_prev[1] + dtt * Lw));
                        }
                    }
                }
            }
            xdu_prev = xdu;
            gyu_prev = gyu;
#pragma unroll
            for (int sk = 0; sk < 2; ++sk) {
                xdd_prev[sk] = xdd[sk];
                gyd_prev[sk] = gyd[sk];
            }
            hat_prev[0] = sH[0][c][lane];
            hat_prev[1] = sH[1][c][lane];
            um = u0; u0 = up; up = u2;
        }
        __syncthreads();  // LDS reuse by the next tile; the stores are visible
        if (mode == MODE_S3) {
            gather_tile_speeds<TU>((const TU*)a.out.u + off_u, (uint32_t)plane, nx, tile.i0, j0,
                                       jend, sch.gas_gamma, smx, smy, sbad);
            __syncthreads();
            if (c == 0) publish_gathered<K>(a, tile.prob, tile.slot, smx, smy, sbad);
        }
    }
}

}  // namespace hweno
