// Fused 2D HWENO stage kernel: reconstruction (Sec. 2.2 Steps 1-3,
// Appendix A), Gauss-point edge values, global Lax-Friedrichs edge fluxes,
// the residual of eq. 2D-semi-discrete-scheme-uniform and the SSP-RK3 stage
// combination with the modified derivatives (Sec. 2.2 Step 4), in one pass.
//
// Work decomposition ("column march"): a workgroup owns a strip of 64
// consecutive columns (60 output columns plus two halo columns per side) and
// marches up through a segment of rows.  Wave c handles conserved component
// c, one column per lane, so the x-neighbours of the stencil come from the
// adjacent lanes and the rows below/above stay in registers as the march
// advances.  Per row:
//   R  each (lane, component) reconstructs its cell and writes the values of
//      U, u_xi, u_eta (local units) at the Gauss points of its four faces to
//      LDS;
//   F  wave k takes one face of every cell (left, right, bottom, top), lane =
//      column, and sums over the face's Gauss points its side of the
//      Lax-Friedrichs flux, all components;
//   S  each (lane, component) adds the two sides of its edges (the x-neighbour's
//      by a lane shift, the lower row's top face from the iteration before) and
//      the dissipation of its average, differences the fluxes of the row below,
//      which now has all four edges, and applies the RK stage to it.
// A face is its own cell's affair, so a wave reads only its own columns, sums
// the Gauss points in registers (with three of them no wave waits for another)
// and hands on one sum instead of a flux per point, in fewer registers than an
// edge point's two sides took: five workgroups instead of four fit a CU in single
// precision (a stage of 2048^2 cells by events 235 -> 225 us in F32_ACC64, 252 ->
// 240 us in F32_KAHAN, 404 us either way in F64; 256^2, Q = 3, F64: 25.6 -> 24.8 us).
// A scalar law has one wave: its face values and fluxes never leave the lane,
// and neither LDS nor a barrier is needed (240^2 Burgers, Q = 3, F64: 15.7 ->
// 11.6 us a stage).
// Both cells of an edge use the same sum of the same numbers, so the update is
// conservative to the rounding of the cell-average arithmetic.
#pragma once

#include "device_common.h"

namespace hweno {

// Gauss-Legendre nodes on [-1/2, 1/2] (ascending) and weights summing to one.
template <int Q> struct Gauss;
template <> struct Gauss<2> {
    static constexpr double g = 0.28867513459481288225;  // 1 / (2 sqrt 3)
    __device__ static constexpr double w(int) { return 0.5; }
};
template <> struct Gauss<3> {
    static constexpr double g = 0.38729833462074168852;  // sqrt(15) / 10
    __device__ static constexpr double w(int mu) { return mu == 1 ? 8.0 / 18.0 : 5.0 / 18.0; }
};

// The same weights for doubled edge fluxes and up to the factor WSUM, which
// goes into 1/dx and 1/dy: the sum over an edge's points costs no product
// (Q = 2) or one.
template <int Q> constexpr double WSUM = Q == 2 ? 0.25 : 5.0 / 36.0;
// Half the weights' sum up to that factor.
template <int Q> constexpr double WHALF = Q == 2 ? 1.0 : 1.8;

// Appendix A coefficients c_{0,1..15} (0..14 here) of the quartic p0 in terms
// of q_1..q_17, written with the centre average subtracted from the nine
// averages (q_5 = 0): every coefficient but the constant is invariant under
// that shift, and the constant becomes relative to the centre.  The march is
// bound by vector instructions (98% of the issue slots in single precision),
// so they come as the numerators n[l] = AN[l] c[l], whose scales go into the
// one product per coefficient that weights p0 below, and the cubic and quartic
// numerators, which are differences of the lower ones, are formed first and
// taken back out of those: 47 instructions instead of 74 for the c themselves.
// (With the blend, face values and edge flux below, 436 instructions a row and
// wave instead of 511, 416 with the faces split over the waves; a stage of 2048^2
// cells 247 -> 235 us in F32_ACC64, 435 -> 404 us in F64.)
constexpr double AN[15] = {2880, 2, 2, 2, 16, 2, 20, 4, 4, 20, 4, 4, 4, 4, 4};
template <class T>
__device__ __forceinline__ void appendix_a(const T* q, T* n) {
    // q[0..16] hold q_1..q_17
    const T S = q[0] + q[2], N = q[6] + q[8], dS = q[2] - q[0], dN = q[8] - q[6];
    const T corner = S + N, ydc = N - S, xdc = dS + dN, xyc = dN - dS;
    const T sx = q[3] + q[5], dxs = q[5] - q[3];
    const T sy = q[1] + q[7], dys = q[7] - q[1];
    const T vWEs = q[9] + q[10], vWEd = q[10] - q[9];
    const T vSNs = q[11] + q[12], vSNd = q[12] - q[11];
    const T wWEs = q[13] + q[14], wWEd = q[14] - q[13];
    const T wSNs = q[15] + q[16], wSNd = q[16] - q[15];
    const T s = sx + sy;
    n[10] = fused((T)-2, sx, vWEd);
    n[14] = fused((T)-2, sy, wSNd);
    n[12] = fused((T)-2, s, corner);
    n[11] = fused((T)-2, vSNd, xyc);
    n[13] = fused((T)-2, wWEd, xyc);
    n[7] = fused((T)-2, dys, ydc);
    n[8] = fused((T)-2, dxs, xdc);
    // 19 dxs - 2 xdc - 6 vWEs + 3 vSNs = 12 dxs - 2 n8 - 3 e, with e the
    // excess of the derivative averages' slope, and so on.  Slopes and curvatures
    // come by the scale that leaves the difference that is most of them exact.
    const T ex = fused((T)2, vWEs, -vSNs) - dxs, ey = fused((T)2, wSNs, -wWEs) - dys;
    n[1] = fused((T)-0.25, ex, fused((T)(-1.0 / 6.0), n[8], dxs));
    n[2] = fused((T)-0.25, ey, fused((T)(-1.0 / 6.0), n[7], dys));
    n[6] = fused((T)2, ex, n[8]);
    n[9] = fused((T)2, ey, n[7]);
    n[3] = fused((T)-0.75, n[10], fused((T)(-1.0 / 24.0), n[12], sx));
    n[5] = fused((T)-0.75, n[14], fused((T)(-1.0 / 24.0), n[12], sy));
    n[4] = fused((T)-5, n[11] + n[13], (T)4 * xyc);
    n[0] = fused((T)81, n[10] + n[14], fused((T)5, n[12], (T)-120 * s));
}

// Nonlinear weights of the 2D blend (eq. nonlinear-weights-2D), as the
// polynomial needs them: with omega_m = gamma_m (1 + tau^2 r_m) / sum and
// r_m = 1 / D_m, omega_0 / gamma_0 = a0 = (1 + tau^2 r_0) / sum and
// omega_m - a0 gamma_m = k d_m, k = tau^2 / sum, d_m = gamma_m (r_m - r_0).
template <class T, bool SQ>
__device__ __forceinline__ void blend_form(const T* beta, const Scheme& s, T& a0, T& k, T* d) {
    const T t = (fabs(beta[0] - beta[1]) + fabs(beta[0] - beta[2])) +
                (fabs(beta[0] - beta[3]) + fabs(beta[0] - beta[4]));
    const T tau = (T)0.25 * t, tau2 = tau * tau;
    const T eps = (T)s.eps;
    T r[5], g[5];
#pragma unroll
    for (int m = 0; m < 5; ++m) {
        r[m] = rcp(SQ ? fused(beta[m], beta[m], eps) : beta[m] + eps);
        g[m] = (T)s.gam[m];
    }
    // the small weights first: added to gamma_0 one by one they leave the sum of
    // the default ones two roundings below 1, which every polynomial would share
    const T gs = ((g[1] + g[2]) + (g[3] + g[4])) + g[0];
    T S = g[0] * r[0];
#pragma unroll
    for (int m = 1; m < 5; ++m) {
        const T gr = g[m] * r[m];
        d[m - 1] = fused(-g[m], r[0], gr);
        S += gr;
    }
    const T inv = rcp(fused(tau2, S, gs));
    a0 = fused(tau2, r[0], (T)1) * inv;
    k = tau2 * inv;
}

// HWENO polynomial of one cell and component (Steps 1-3).  q: stencil with
// the centre average subtracted.  C: coefficients of u_ij - u-bar_ij in the
// basis 1, X, Y, X^2, X Y, Y^2, X^3, X^2 Y, X Y^2, Y^3, X^4, X^3 Y, X^2 Y^2,
// X Y^3, Y^4 with X = 2 xi, Y = 2 eta, so that the faces lie at +-1 and the
// face values below need no powers of one half.
template <class T>
__device__ __forceinline__ void reconstruct2d(const T* q, const Scheme& s, int squared, T* C,
                                              T& vhat, T& what) {
    T n[15];
    appendix_a(q, n);
    // linear polynomials on the L-shaped stencils S1..S4: slopes only
    const T sW = -q[3], sE = q[5], sS = -q[1], sN = q[7];
    T beta[5];
    if (s.smoothness == BETA_CLASSICAL) {
        T c0[15];
#pragma unroll
        for (int l = 0; l < 15; ++l) c0[l] = n[l] * (T)(1.0 / AN[l]);
        beta[0] = beta_classical_2d(c0);
    } else {
        // smoothness indicator: sum over monomials of (m! n! c_mn)^2
        auto sq2 = [](T a, T b) { return fused(a, a, b * b); };
        T b0 = fused(n[3], n[3], fused(n[5], n[5], n[12] * n[12]));   // 4 c3^2, 4 c5^2, 16 c12^2
        b0 = fused((T)0.25, sq2(n[1], n[2]), b0);
        b0 = fused((T)(1.0 / 256.0), n[4] * n[4], b0);
        b0 = fused((T)0.09, sq2(n[6], n[9]), b0);
        b0 = fused((T)0.25, sq2(n[7], n[8]), b0);
        b0 = fused((T)2.25, sq2(n[11], n[13]), b0);
        beta[0] = fused((T)36, sq2(n[10], n[14]), b0);
    }
    const T sW2 = sW * sW, sE2 = sE * sE;
    beta[1] = fused(sS, sS, sW2);
    beta[2] = fused(sS, sS, sE2);
    beta[3] = fused(sN, sN, sE2);
    beta[4] = fused(sN, sN, sW2);
    // u_ij = w0/g0 p0 + sum_m (w_m - w0 g_m/g0) p_m   (eq. hweno-reconstruction-2D)
    T a0 = (T)1, k = (T)0, d[4] = {0, 0, 0, 0};
    if (s.weights != W_LINEAR) {
        if (squared) blend_form<T, true>(beta, s, a0, k, d);
        else blend_form<T, false>(beta, s, a0, k, d);
    }
    // coefficient l of p0 is n[l] / AN[l], in X and Y divided by 2^degree
    const T w64 = a0 * (T)(1.0 / 64.0), w32 = a0 * (T)(1.0 / 32.0), w160 = a0 * (T)(1.0 / 160.0);
    const T w8 = a0 * (T)0.125, w4 = a0 * (T)0.25, kh = (T)0.5 * k;
    C[0] = a0 * (T)(1.0 / 2880.0) * n[0];
    C[1] = fused(kh, fused(sW, d[0] + d[3], sE * (d[1] + d[2])), w4 * n[1]);
    C[2] = fused(kh, fused(sS, d[0] + d[1], sN * (d[2] + d[3])), w4 * n[2]);
    C[3] = w8 * n[3];
    C[5] = w8 * n[5];
    C[6] = w160 * n[6];
    C[9] = w160 * n[9];
    C[7] = w32 * n[7];
    C[8] = w32 * n[8];
    C[4] = w64 * n[4];
#pragma unroll
    for (int l = 10; l < 15; ++l) C[l] = w64 * n[l];
    // modified derivatives: integrals of u_x, u_y over the cell (scaled units)
    vhat = fused((T)2, C[1] + C[6], (T)(2.0 / 3.0) * C[8]);
    what = fused((T)2, C[2] + C[9], (T)(2.0 / 3.0) * C[7]);
}

// Values at the Gauss points of the two faces normal to the first variable
// of C (X for x-faces; pass the transposed coefficients for y-faces).
// Outputs per side s (0: -1, 1: +1) and node mu: value, derivative normal to
// the face, derivative along the face (by X and Y: half of the derivatives by
// xi and eta; relative value).  Parities in the two variables: E, O even and
// odd parts in the normal one at the face, by powers of the other; then ee,
// oe, eo, oo by both.  An odd part's last factor goes into the sum that
// combines the parts.  half: half the sum of a side's values, with the points'
// weights up to WSUM.
template <class T, int Q>
__device__ __forceinline__ void face_values(const T* C, T (*val)[Q], T (*dn)[Q], T (*dt)[Q],
                                            T* half) {
    const T E0 = C[0] + (C[3] + C[10]), O0 = C[1] + C[6];
    const T E1 = C[2] + C[7], O1 = C[4] + C[11];
    const T E2 = C[5] + C[12], O2 = C[8];
    const T E3 = C[9], O3 = C[13];
    const T E4 = C[14];
    const T Eb0 = fused((T)3, C[6], C[1]), Ob0 = fused((T)2, C[10], C[3]);   // Ob: half of the odd parts
    const T Eb1 = fused((T)3, C[11], C[4]), Ob1 = C[7];
    const T Eb2 = C[8], Ob2 = C[12];
    const T Eb3 = C[13];
    constexpr double gd = 2.0 * Gauss<Q>::g;   // nodes at +-g in [-1, 1]
    const T g = (T)gd, g2 = (T)(gd * gd);
    const T uee = fused(g2, fused(g2, E4, E2), E0), uoe = fused(g2, O2, O0);
    const T ueo = fused(g2, E3, E1), uoo = fused(g2, O3, O1);             // times g
    const T nee = fused(g2, Eb2, Eb0), noe = fused(g2, Ob2, Ob0);         // noe times 2
    const T neo = fused(g2, Eb3, Eb1), noo = Ob1;                         // times g, 2 g
    const T tee = fused((T)(3.0 * gd * gd), E3, E1), toe = fused((T)(3.0 * gd * gd), O3, O1);
    const T teo = fused((T)(2.0 * gd * gd), E4, E2), too = O2;            // times 2 g
    constexpr int lo = 0, hi = Q - 1;  // nodes -g and +g
#pragma unroll
    for (int s = 0; s < 2; ++s) {
        const T sg = s ? (T)1 : (T)-1;
        const T ue = uee + sg * uoe, uo = ueo + sg * uoo;
        const T ne = fused((T)2 * sg, noe, nee), no = fused((T)2 * sg, noo, neo);
        const T te = tee + sg * toe, to = teo + sg * too;
        val[s][lo] = fused(-g, uo, ue); val[s][hi] = fused(g, uo, ue);
        dn[s][lo] = fused(-g, no, ne);  dn[s][hi] = fused(g, no, ne);
        dt[s][lo] = fused((T)-2 * g, to, te); dt[s][hi] = fused((T)2 * g, to, te);
        if (Q == 3) {
            val[s][1] = E0 + sg * O0;
            dn[s][1] = fused((T)2 * sg, Ob0, Eb0);
            dt[s][1] = E1 + sg * O1;
        }
        half[s] = Q == 2 ? ue : fused((T)0.8, val[s][1], ue);
    }
}

template <class T> __device__ __forceinline__ void transpose15(const T* C, T* D) {
    D[0] = C[0]; D[1] = C[2]; D[2] = C[1]; D[3] = C[5]; D[4] = C[4]; D[5] = C[3];
    D[6] = C[9]; D[7] = C[8]; D[8] = C[7]; D[9] = C[6]; D[10] = C[14]; D[11] = C[13];
    D[12] = C[12]; D[13] = C[11]; D[14] = C[10];
}

// One side of the Lax-Friedrichs flux at a face's Gauss point, TWICE its value:
// f(U), and of the derivative fluxes also al times their argument (al = alpha
// for a cell's right or top face, -alpha for its left or bottom one); the 1/2 is
// folded into the residual's factors.  FIRST starts the sum over the points.
// ld(v, D): the face's values of kind v.
//
// The dissipation alpha (U_L - U_R) of the averages is left out here and taken
// from the values relative to the cells' averages and the averages' difference:
// a side's alpha U, summed over the points before the other side is taken off,
// would be rounded at the size of alpha U, whose difference across the edge is
// of fifth order.
template <bool FIRST, class T, int FLUX, int K, int DIR, class LD>
__device__ __forceinline__ void lf_side(const Flux<T, FLUX, K, DIR>& F, T al, LD ld, T* out) {
    if constexpr (FLUX == F_EULER && K == 4) {
        T D[K];
        ld(0, D);
        const auto w = F.prim(D, al);
        F.template flux<FIRST>(D, w, out);
#pragma unroll
        for (int v = 1; v < 3; ++v) {
            ld(v, D);
            F.template jvp<FIRST>(D, w, al, out + v * K);
        }
    } else {
        T U[K], V[K], W[K], f[K], fv[K], fw[K];
        ld(0, U);
        ld(1, V);
        ld(2, W);
        F.side(U, V, W, f, fv, fw);
#pragma unroll
        for (int c = 0; c < K; ++c) {
            out[c] = FIRST ? f[c] : out[c] + f[c];
            out[K + c] = fused(al, V[c], FIRST ? fv[c] : out[K + c] + fv[c]);
            out[2 * K + c] = fused(al, W[c], FIRST ? fw[c] : out[2 * K + c] + fw[c]);
        }
    }
}
// The sum over a face's points, up to the factor WSUM.  ld(mu, v, D).
template <int Q, class T, int FLUX, int K, int DIR, class LD>
__device__ __forceinline__ void lf_face(const Flux<T, FLUX, K, DIR>& F, T al, LD ld, T* out) {
    auto at = [&](int mu) { return [&ld, mu](int v, T* D) { ld(mu, v, D); }; };
    if constexpr (Q == 2) {
        lf_side<true>(F, al, at(0), out);
        lf_side<false>(F, al, at(1), out);
    } else {
        lf_side<true>(F, al, at(1), out);
#pragma unroll
        for (int k = 0; k < 3 * K; ++k) out[k] *= (T)1.6;
        lf_side<false>(F, al, at(0), out);
        lf_side<false>(F, al, at(2), out);
    }
}

// One wave: the maxima that gather_tile_speeds left and the end of the tile's step.
template <int K>
__device__ __forceinline__ void publish_gathered(const StageArgs& a, int prob, int slot,
                                                 const double* smx, const double* smy,
                                                 const long long* sbad) {
    double mx = smx[0], my = smy[0];
    long long bad = sbad[0];
#pragma unroll
    for (int v = 1; v < K; ++v) {
        mx = fmax(mx, smx[v]);
        my = fmax(my, smy[v]);
        bad = min(bad, sbad[v]);
    }
    publish_and_end(&a.probs[prob], prob, slot, a.ctl, a.flags, 1, mx, my, bad);
}

// Waves per SIMD the register allocation must allow (launch bounds); for the
// four-wave Euler workgroups also workgroups per CU.  Variant 0: what registers
// and the LDS of the faces allow without spilling (the face sums take one side and
// quantity at a time and stage 3's speed gather is a call of its own after the
// march: at most 96 registers in single precision with two Gauss points, 103 with
// three, 144 and 170 in FP64); variant 1 (stage2d_two_variants): one more, which
// caps the registers lower (the compiler spills).  The tuner picks.  The one-wave
// scalar laws use no LDS; in FP64 they take up to 191 registers.
template <int P, int K, int Q, int V> constexpr int stage2d_min_waves() {
    return K == 1 ? (P == P_F64 ? 2 : 4) : stage2d_slots(P, true, Q, false) + V;
}

template <int P, int K, int Q, int FLUX, int mode, int V>
__global__ void __launch_bounds__(64 * K, (stage2d_min_waves<P, K, Q, V>())) stage2d_kernel(StageArgs a) {
    using TU = typename PrecT<P>::TU;
    using TD = typename PrecT<P>::TD;
    using T = typename PrecT<P>::T;
    using TA = typename PrecT<P>::TA;
    // Values of the four faces (left, right, bottom, top) at their Gauss
    // points, entry (mu*3 + v)*K + comp, v = value, d/dX, d/dY.  A face's
    // side of the flux, entry sk*K + comp (sk = u, v, w flux), is written over
    // them: only the thread of that face and column reads its values, and it
    // reads them all before it writes; the residual of component c reads only
    // entries of component c, which the next row's reconstruction rewrites in
    // the same wave, so no other wave can overwrite a flux before it is read.
    constexpr bool SHARE = K > 1;
    __shared__ T sF[SHARE ? 4 : 1][SHARE ? Q * 3 * K : 1][64];
    __shared__ double smx[K], smy[K];  // stage 3: per-wave maxima of the wave speeds
    __shared__ long long sbad[K];      // stage 3: per-wave first non-admissible cell
    constexpr bool S3 = mode == MODE_S3;
    // The RK inputs of the output row are loaded before the reconstruction, or, by
    // the Euler kernels with wide averages and single-precision faces, before the
    // faces, which are long enough for them to arrive: through the reconstruction
    // they would hold four registers that do not fit the 96 of five workgroups a
    // CU (8 to 32 bytes of scratch and 2 to 3% of a stage of 2048^2 cells in
    // F32_ACC64).  In F32, where they fit, late loads cost 2%.
    constexpr bool LATE_RK = K > 1 && sizeof(T) == 4 && sizeof(TU) == 8;

    const int lane = threadIdx.x & 63;
    // component of this wave (uniform: the plane pointers stay in SGPRs)
    const int c = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const Scheme& sch = a.sch;
    const int squared = sch.weights == W_BETA2 || (sch.weights == W_PAPER);
    const Flux<T, FLUX, K, 0> FXf(sch);
    const Flux<T, FLUX, K, 1> FYf(sch);
    const Tile2D* tiles = (const Tile2D*)a.tiles + a.tile_offset;

    // Stage 3 also gathers the wave speeds of the state it writes (for the
    // next step's flux and time step).  A scalar law's are taken from the
    // value as it is written.  For Euler the tile's new averages are read back
    // after its march by every wave (they are in the caches the stores went
    // through), so the march itself carries no extra registers: passing each
    // row through LDS to one wave inside the march was 320 us a stage instead
    // of 250 at 2048^2 in F32_ACC64 and 451 instead of 423 in F64.

    for (int tix = blockIdx.x; tix < a.ntiles; tix += gridDim.x) {
        const Tile2D tile = tiles[tix];
        const ProbDev& P_ = a.probs[tile.prob];
        StepChoice step{};
        if (mode != MODE_RHS) {
            step = stage_step(P_, a.ctl, a.flags, mode);
            if (!step.act) {
                if (mode == MODE_S3 && threadIdx.x < 64)
                    publish_and_end(&a.probs[tile.prob], tile.prob, tile.slot, a.ctl, a.flags, 0,
                                    0.0, 0.0, LLONG_MAX);
                continue;
            }
        }
        const int nx = P_.nx, ny = P_.ny, bcx = P_.bc_x, bcy = P_.bc_y;
        const int64_t plane = (int64_t)nx * ny;
        // the residual's factors, with the edge sums' weight; the derivatives
        // at the edge points are by X = 2 xi, Y = 2 eta
        const T inv_dx = (T)(P_.inv_dx * (2.0 * WSUM<Q>)), inv_dy = (T)(P_.inv_dy * (2.0 * WSUM<Q>));
        const TA inv_dx_a = (TA)(P_.inv_dx * WSUM<Q>), inv_dy_a = (TA)(P_.inv_dy * WSUM<Q>);
        const T rx = (T)(P_.dx * P_.inv_dy), ry = (T)(P_.dy * P_.inv_dx);
        const T ax = (T)as_double(P_.ax_bits), ay = (T)as_double(P_.ay_bits);
        const double dt = step.dt;
        const int gi = tile.i0 - 2 + lane;          // this lane's column
        const int li = bc_map(gi, nx, bcx);         // column it reads
        const bool out_col = lane >= 2 && lane < 62 && gi < nx;

        // Every pointer of the march is formed here, once per tile: fields of
        // the problem table read inside the row loop would be reloaded after
        // each store (possible aliasing) and waited for with every load in
        // flight, the row-ahead prefetch included.
        const int64_t off_u = P_.off_u, off_d = P_.off_d;
        const TU* Uu = (const TU*)a.in.u + off_u + c * plane;
        const TD* Uv = (const TD*)a.in.d + off_d + c * plane;
        const TD* Uw = (const TD*)a.in.d + off_d + (K + c) * plane;
        const TU* Un = (const TU*)a.un + off_u + c * plane;     // stages 2, 3: U^n
        TD* Hv = (TD*)a.h + off_d + c * plane;                  // saved derivatives
        TD* Hw = (TD*)a.h + off_d + (K + c) * plane;
        TU* Ou = (TU*)a.out.u + off_u + c * plane;
        TD* Ov = (TD*)a.out.d + off_d + c * plane;
        TD* Ow = (TD*)a.out.d + off_d + (K + c) * plane;

        auto row_ptr = [&](int j) { return (uint32_t)(bc_map(j, ny, bcy) * nx + li); };
        // Solid walls: in a mirror image across x the x momentum (component
        // 1) is odd and the other averages even, and v-bar has the opposite
        // parity of its quantity; across y likewise with component 2 and
        // w-bar.  Signs of this lane's column, and of a row.
        const bool mx = FLUX == F_EULER && wall_mirrored(gi, nx, bcx);
        const bool nux = mx && c == 1, nvx = mx && c != 1, nwx = mx && c == 1;
        auto load_row = [&](int j, TU& u, TD& v, TD& w) {
            const uint32_t o = row_ptr(j);
            const bool my = FLUX == F_EULER && wall_mirrored(j, ny, bcy);
            const bool nuy = my && c == 2, nvy = my && c == 2, nwy = my && c != 2;
            u = neg_if(plane_at(Uu, o), nux != nuy);
            v = neg_if(plane_at(Uv, o), nvx != nvy);
            w = neg_if(plane_at(Uw, o), nwx != nwy);
        };
        const int j0 = tile.j0, jend = tile.j0 + tile.nrows;  // outputs j0..jend-1

        TU um, u0, up, un_;
        TD vm, v0, vp, vn_, wm, w0, wp, wn_;
        load_row(j0 - 2, um, vm, wm);
        load_row(j0 - 1, u0, v0, w0);
        load_row(j0, up, vp, wp);
        constexpr bool SYMD = sizeof(T) == 4 && (std::is_same<TU, double>::value || std::is_same<TU, float>::value);
        T dneg = 0;
        if constexpr (SYMD) dneg = (T)(u0 - um);
        T top_prev[3] = {0, 0, 0};   // the previous row's top sides (this lane, comp)
        // previous row's flux sums: x differences and y sums of the
        // cell-average fluxes in the accumulation type, of the derivative
        // fluxes in T.  The FP64 path (PARTIAL) carries instead the part of
        // the previous row's residual known before its top edge (its x
        // difference less its bottom edge, in xdu_prev and xdd_prev): three
        // register pairs fewer through the march.  (In single precision
        // that form would round the sum of two large terms instead of their
        // small difference.)
        constexpr bool PARTIAL = P == P_F64;
        TA xdu_prev = 0, gyu_prev = 0;
        T xdd_prev[2] = {0, 0}, gyd_prev[2] = {0, 0};
        T hat_prev[2] = {0, 0};

        double mxl = 0.0, myl = 0.0;     // stage 3 of a scalar law: this lane's maxima
        long long badl = LLONG_MAX;
        for (int r = j0 - 1; r <= jend; ++r) {
            // prefetch the row two above
            load_row(r + 2, un_, vn_, wn_);
            TA unr = 0;
            T hvr = 0, hwr = 0;
            const bool emit = r > j0 && out_col;   // row r-1 is an output row
            const uint32_t oo = (uint32_t)((r - 1) * nx + gi);  // output row r-1 (in range if emit)
            auto load_rk = [&]() {
                // unconditional (lanes without output read element 0) so that
                // the loads stay in flight until the epilogue uses them
                const uint32_t ol = emit ? oo : 0u;
                unr = (TA)plane_at(Un, ol);
                hvr = (T)plane_at(Hv, ol);
                hwr = (T)plane_at(Hw, ol);
            };
            if constexpr ((mode == MODE_S2 || mode == MODE_S3) && !LATE_RK) load_rk();

            // ---- R: reconstruct cell (gi, r), component c -------------------
            T q[17];
            if constexpr (sizeof(T) == 4) {
                // Single precision: the column's own differences and the
                // differences of the side neighbours' averages from the centre
                // are rounded once from the wide averages; a corner is the sum
                // of the neighbour column's own difference and that column's
                // centre difference, which the compiler forms in one add with a
                // DPP lane shift on its first operand.
                const TU uc = u0;
                const T dp = (T)(up - uc), dr = (T)(from_right(u0) - uc);
                T dm, dl;
                if constexpr (SYMD) {
                    dm = -dneg;
                    dl = -from_left(dr);
                    dneg = dp;
                } else {
                    dm = (T)(um - uc);
                    dl = (T)(from_left(u0) - uc);
                }
                q[0] = from_left(dm) + dl;
                q[1] = dm;
                q[2] = from_right(dm) + dr;
                q[3] = dl;
                q[4] = (T)0;
                q[5] = dr;
                q[6] = from_left(dp) + dl;
                q[7] = dp;
                q[8] = from_right(dp) + dr;
            } else {
                const TU uc = u0;
                q[0] = (T)(from_left(um) - uc);
                q[1] = (T)(um - uc);
                q[2] = (T)(from_right(um) - uc);
                q[3] = (T)(from_left(u0) - uc);
                q[4] = (T)0;
                q[5] = (T)(from_right(u0) - uc);
                q[6] = (T)(from_left(up) - uc);
                q[7] = (T)(up - uc);
                q[8] = (T)(from_right(up) - uc);
            }
            {
                q[9] = (T)from_left(v0);
                q[10] = (T)from_right(v0);
                q[11] = (T)vm;
                q[12] = (T)vp;
                q[13] = (T)from_left(w0);
                q[14] = (T)from_right(w0);
                q[15] = (T)wm;
                q[16] = (T)wp;
            }
            T C[15], vhat, what;
            reconstruct2d<T>(q, sch, squared, C, vhat, what);
            const T ucT = (T)u0;
            // the rows beside the segment only lend it an edge: their x faces
            // and far y faces are left out
            const bool inner = r >= j0 && r < jend;
            T FV[4][Q][3];   // a scalar law's face values
            auto put = [&](int f, const T (*val)[Q], const T (*dX)[Q], const T (*dY)[Q]) {
#pragma unroll
                for (int mu = 0; mu < Q; ++mu)
#pragma unroll
                    for (int v = 0; v < 3; ++v) {
                        const T x = v == 0 ? ucT + val[f & 1][mu] : (v == 1 ? dX : dY)[f & 1][mu];
                        if constexpr (SHARE) sF[f][(mu * 3 + v) * K + c][lane] = x;
                        else FV[f][mu][v] = x;
                    }
            };
            // Derivatives go to the faces in local units (d/dX, d/dY): the
            // edge flux is linear in them, so the 2/dx, 2/dy of u_x, u_y are
            // applied once to the residual instead of at every face point.
            T val[2][Q], dn[2][Q], dtg[2][Q], half[2];
            // The dissipation of the averages, alpha (U_L - U_R) over the points:
            // jump_x at the right edge (unused beside the segment); the bottom
            // edge's goes onto the side of the row below.
            T jump_x = q[5], half_top;
            if (inner) {
                face_values<T, Q>(C, val, dn, dtg, half);   // x-faces: dn = d/dX, dt = d/dY
                put(0, val, dn, dtg);
                put(1, val, dn, dtg);
                jump_x = fused((T)-WHALF<Q>, q[5], half[1] - from_right(half[0]));
            }
            {
                T D[15];
                transpose15(C, D);
                face_values<T, Q>(D, val, dn, dtg, half);   // y-faces: dn = d/dY, dt = d/dX
                put(2, val, dtg, dn);
                put(3, val, dtg, dn);
                const T jump_y = fused((T)WHALF<Q>, q[1], -half[0]);
                top_prev[0] = fused(ay, jump_y + jump_y, top_prev[0]);
                half_top = half[1];
            }

            if constexpr ((mode == MODE_S2 || mode == MODE_S3) && LATE_RK) load_rk();

            // ---- F: the faces' sides of the edge fluxes ---------------------
            T side[4][3];   // of this lane's cell, this component
            if constexpr (SHARE) {
                __syncthreads();  // A: face values of row r ready
                auto face = [&](auto fi, const auto& F, T al) {
                    constexpr int f = decltype(fi)::value;
                    T out[3 * K];
                    lf_face<Q>(F, al, [&](int mu, int v, T* D) {
#pragma unroll
                        for (int k = 0; k < K; ++k) D[k] = sF[f][(mu * 3 + v) * K + k][lane];
                    }, out);
#pragma unroll
                    for (int k = 0; k < 3 * K; ++k) sF[f][k][lane] = out[k];
                };
                if (inner || c == (r < j0 ? 3 : 2)) {
                    if (c == 0) face(std::integral_constant<int, 0>(), FXf, -ax);
                    else if (c == 1) face(std::integral_constant<int, 1>(), FXf, ax);
                    else if (c == 2) face(std::integral_constant<int, 2>(), FYf, -ay);
                    else face(std::integral_constant<int, 3>(), FYf, ay);
                }
                __syncthreads();  // B: fluxes ready
#pragma unroll
                for (int f = 0; f < 4; ++f)
#pragma unroll
                    for (int sk = 0; sk < 3; ++sk) side[f][sk] = sF[f][sk * K + c][lane];
            } else {
                auto face = [&](int f, const auto& F, T al) {
                    lf_face<Q>(F, al, [&](int mu, int v, T* D) { D[0] = FV[f][mu][v]; }, side[f]);
                };
#pragma unroll
                for (int sk = 0; sk < 3; ++sk) side[0][sk] = side[1][sk] = 0;
                if (inner) {
                    face(0, FXf, -ax);
                    face(1, FXf, ax);
                }
                face(2, FYf, -ay);
                face(3, FYf, ay);
            }
            // ---- S: residual and RK stage of row r-1 ------------------------
            // The derivative fluxes are differenced in T: the difference of
            // two T values rounded to T is what a wider difference rounds to.
            {
                TA xdu = 0, gyu = 0;
                T xdd[2], gyd[2];
#pragma unroll
                for (int sk = 0; sk < 3; ++sk) {
                    T fr = side[1][sk] + from_right(side[0][sk]);         // right edge
                    if (sk == 0) fr = fused(ax, jump_x + jump_x, fr);
                    const T fl = from_left(fr);                           // left edge
                    const T g = top_prev[sk] + side[2][sk];               // edge to row r-1
                    top_prev[sk] = sk == 0 ? fused(ay, half_top + half_top, side[3][sk]) : side[3][sk];
                    if (sk == 0) {
                        xdu = (TA)fr - (TA)fl;
                        gyu = (TA)g;
                    } else {
                        xdd[sk - 1] = fr - fl;
                        gyd[sk - 1] = g;
                    }
                }
                if (r > j0) {
                    // v- and w-fluxes carry the derivatives in local units
                    TA Lu;
                    T Lv, Lw;
                    if constexpr (PARTIAL) {
                        Lu = -(xdu_prev + gyu * inv_dy_a);
                        Lv = -inv_dx * (xdd_prev[0] + rx * gyd[0]);
                        Lw = -inv_dy * (xdd_prev[1] + gyd[1]);
                    } else {
                        Lu = -(xdu_prev * inv_dx_a + (gyu - gyu_prev) * inv_dy_a);
                        Lv = -inv_dx * (xdd_prev[0] + rx * (gyd[0] - gyd_prev[0]));
                        Lw = -inv_dy * (ry * xdd_prev[1] + (gyd[1] - gyd_prev[1]));
                    }
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
                                const TU nu = (TU)(third * unr + two3 * (ucur + dta * Lu));
                                plane_at(Ou, oo) = nu;
                                if constexpr (!SHARE) {
                                    const double w = (double)nu;
                                    double sx, sy;
                                    if (wave_speed<FLUX, 2, K>(&w, sch, sx, sy)) {
                                        mxl = fmax(mxl, sx);
                                        myl = fmax(myl, sy);
                                    } else {
                                        badl = min(badl, (long long)oo);
                                    }
                                }
                                plane_at(Ov, oo) = (TD)((T)(1.0 / 3.0) * hvr +
                                              (T)(2.0 / 3.0) * (hat_prev[0] + dtt * Lv));
                                plane_at(Ow, oo) = (TD)((T)(1.0 / 3.0) * hwr +
                                              (T)(2.0 / 3.0) * (hat_prev[1] + dtt * Lw));
                            }
                        }
                    }
                }
                if constexpr (PARTIAL) {
                    xdu_prev = xdu * inv_dx_a - gyu * inv_dy_a;
                    xdd_prev[0] = xdd[0] - rx * gyd[0];
                    xdd_prev[1] = ry * xdd[1] - gyd[1];
                } else {
                    xdu_prev = xdu;
                    gyu_prev = gyu;
#pragma unroll
                    for (int sk = 0; sk < 2; ++sk) {
                        xdd_prev[sk] = xdd[sk];
                        gyd_prev[sk] = gyd[sk];
                    }
                }
            }
            hat_prev[0] = vhat;
            hat_prev[1] = what;
            // advance the register window one row up
            um = u0; u0 = up; up = un_;
            vm = v0; v0 = vp; vp = vn_;
            wm = w0; w0 = wp; wp = wn_;
        }
        if constexpr (SHARE) __syncthreads();  // LDS reuse by the next tile; the stores are visible
        if constexpr (S3) {
            if constexpr (SHARE) {
                gather_tile_speeds<TU>((const TU*)a.out.u + off_u, (uint32_t)plane, nx, tile.i0, j0,
                                       jend, sch.gas_gamma, smx, smy, sbad);
                __syncthreads();
            } else {
                mxl = wave_max_d(mxl);
                myl = wave_max_d(myl);
                if (__any(badl != LLONG_MAX)) badl = wave_min_ll(badl);
            }
            if (threadIdx.x < 64) {
                // the tile is read again rather than held through the march
                const volatile Tile2D* t = &tiles[tix];
                const int prob = t->prob, slot = t->slot;
                if constexpr (SHARE) publish_gathered<K>(a, prob, slot, smx, smy, sbad);
                else publish_and_end(&a.probs[prob], prob, slot, a.ctl, a.flags, 1, mxl, myl, badl);
            }
        }
    }
}

// Launches the stage kernel of one precision: Euler in either register variant
// where there are two, the scalar laws in variant 0.
template <int P, int K, int Q, int FLUX, int V>
void stage2d_launch_modes(int mode, const StageArgs& a, int grid, hipStream_t s) {
    constexpr int threads = 64 * K;
    switch (mode) {
        case MODE_RHS: stage2d_kernel<P, K, Q, FLUX, MODE_RHS, V><<<grid, threads, 0, s>>>(a); break;
        case MODE_S1: stage2d_kernel<P, K, Q, FLUX, MODE_S1, V><<<grid, threads, 0, s>>>(a); break;
        case MODE_S2: stage2d_kernel<P, K, Q, FLUX, MODE_S2, V><<<grid, threads, 0, s>>>(a); break;
        default: stage2d_kernel<P, K, Q, FLUX, MODE_S3, V><<<grid, threads, 0, s>>>(a); break;
    }
}

template <int P, int Q>
void stage2d_launch_euler(int mode, int variant, const StageArgs& a, int grid, hipStream_t s) {
    if constexpr (stage2d_two_variants(P, true, Q, false)) {
        if (variant) return stage2d_launch_modes<P, 4, Q, F_EULER, 1>(mode, a, grid, s);
    }
    stage2d_launch_modes<P, 4, Q, F_EULER, 0>(mode, a, grid, s);
}

template <int P>
hipError_t stage2d_launch_prec(int flux, int Q, int mode, int variant, const StageArgs& a,
                               int grid, hipStream_t s) {
    if (flux == F_EULER) {
        if (Q == 2) stage2d_launch_euler<P, 2>(mode, variant, a, grid, s);
        else stage2d_launch_euler<P, 3>(mode, variant, a, grid, s);
    } else if (flux == F_BURGERS) {
        if (Q == 2) stage2d_launch_modes<P, 1, 2, F_BURGERS, 0>(mode, a, grid, s);
        else stage2d_launch_modes<P, 1, 3, F_BURGERS, 0>(mode, a, grid, s);
    } else {
        if (Q == 2) stage2d_launch_modes<P, 1, 2, F_ADV, 0>(mode, a, grid, s);
        else stage2d_launch_modes<P, 1, 3, F_ADV, 0>(mode, a, grid, s);
    }
    return hipGetLastError();
}

}  // namespace hweno
