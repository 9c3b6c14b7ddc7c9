// cns_device.h -- device arithmetic of the WENO5-Roe / central-viscous discretisation
// for gfx950, FP64 (the mixed form's FP32 arithmetic is in cns_mixed.hip, which shares the
// reciprocals and the central difference).
//
// Formulation choices (same operator as Sec. 2.2 of the paper, different
// arithmetic order):
//  * WENO5 by cells: the indicators of a cell serve the left-biased value at its right
//    face and the right-biased value at its left face (weno5_cell6).
//  * Nonlinear weights: alpha_k = c_k / d_k with d_k = (eps + beta_k)^2 are scaled by
//    d_1 d_2 d_3, so a normalisation needs one division.
//  * The sweeps carry 6 x the reconstructed values and 4 x the indicators (with 4 eps),
//    which removes the constant factors from the inner arithmetic; the interface flux
//    divides once by 12 at the end.
//  * Nine reconstructions per direction instead of ten: the mass flux is the momentum
//    along the line.
//  * Roe dissipation |A| (u^R - u^L) is evaluated with wave strengths (projections
//    on the left eigenvectors, written out) instead of explicit 5x5 matrices;
//    |A| = X |Lambda| X^-1 is basis independent so the operator is the same.
#pragma once
#include <hip/hip_runtime.h>

#include "cns.h"

namespace cns {

struct PhysT {
    double gamma, prandtl, mu_eff, eps, delta;
};

// Reciprocal: the hardware estimate r (relative error below 2^-24 on gfx950, measured)
// refined once to third order, 1/b = r / (1 - e) ~ r (1 + e + e^2) with e = 1 - b r
// (truncation e^3 < 2^-72), three instructions against four for two Newton-Raphson
// steps; in FP32 one Newton-Raphson step r <- r + r e.  Within an ulp or two of the
// IEEE division, at about half its instructions.
__device__ __forceinline__ double rcp(double b) {
    const double r = __builtin_amdgcn_rcp(b);
    const double e = fma(-b, r, 1.0);
    return fma(r, fma(e, e, e), r);
}
__device__ __forceinline__ float rcp(float b) {
    float r = __builtin_amdgcn_rcpf(b);
    float e = fmaf(-b, r, 1.0f);
    return fmaf(r, e, r);
}

// Reciprocal square root: the hardware estimate y (relative error below 2^-24) refined
// once to third order, x^-1/2 = y (1 - e)^-1/2 ~ y (1 + e/2 + 3 e^2 / 8) with
// e = 1 - x y^2 (truncation 5 e^3 / 16); in FP32 one Newton-Raphson step
// y <- y + y e / 2.
__device__ __forceinline__ double rsq(double x) {
#pragma clang fp contract(off)
    const double y = __builtin_amdgcn_rsq(x);
    const double e = fma(-x * y, y, 1.0);
    return fma(y * e, fma(e, 0.375, 0.5), y);
}
__device__ __forceinline__ float rsq(float x) {
#pragma clang fp contract(off)
    float y = __builtin_amdgcn_rsqf(x);
    float r = fmaf(-x * y, y, 1.0f);
    return fmaf(0.5f * y, r, y);
}

// Harten's entropy fix: |lam| if |lam| >= delta, else (lam^2 + delta^2) h, h = 1 / (2 delta)
template <typename T>
__device__ __forceinline__ T harten_abs(T lam, T delta, T h) {
#pragma clang fp contract(off)
    T a = fabs(lam);
    return (a >= delta) ? a : (lam * lam + delta * delta) * h;
}

// Holds a value at this point of the program: pure arithmetic whose result is only used in
// a later block would otherwise be sunk into that block, past the scheduling fences that
// bound what is live.
template <typename T>
__device__ __forceinline__ void pin(T &v) {
    asm volatile("" : "+v"(v));
}

__device__ __forceinline__ double fmadd(double a, double b, double c) { return fma(a, b, c); }
__device__ __forceinline__ float fmadd(float a, float b, float c) { return fmaf(a, b, c); }

// The functions from here to the interface flux state every fused multiply-add
// themselves (contraction off): an interface flux has the same bits wherever and in
// whichever kernel it is formed, so results do not depend on segment lengths, chunks,
// unrolling or the compiler's choice of what to fuse.

// ---------------------------------------------------------------------------
// WENO5 by cells.  The left-biased value at j+1/2 and the right-biased one at j-1/2 are
// both evaluated from the three parabolas of cell j (stencils j-2..j, j-1..j+1, j..j+2)
// with the same smoothness indicators; only the optimal weights (1, 6, 3)/10 and
// (3, 6, 1)/10 and the candidates are mirrored.  A cell's indicators, their squares and
// products are therefore formed once for the two interfaces that share them (an
// evaluation by interface forms them for each bias: 55 instead of 74 FP64 operations per
// left/right pair).  Everything is formed from the differences g_i of the stencil, the
// values as 6 q_j plus a correction, six times the plain values.
// ---------------------------------------------------------------------------
// The mapped weights of Henrick et al. (2005): the Jiang-Shu weights w (optimal values
// 1/10, 6/10, 3/10) passed through g_k(w) = w (c_k + c_k^2 - 3 c_k w + w^2) / (c_k^2 + w (1 -
// 2 c_k)), scaled by the product of the three denominators; returns their sum.
__device__ __forceinline__ double weno_map(double w1, double w2, double w3, double g[3]) {
#pragma clang fp contract(off)
    const double N1 = w1 * fmadd(w1, w1 - (0.3), (0.1 + 0.1 * 0.1)), D1 = fmadd(w1, (0.8), (0.1 * 0.1));
    const double N2 = w2 * fmadd(w2, w2 - (1.8), (0.6 + 0.6 * 0.6)), D2 = fmadd(w2, (-0.2), (0.6 * 0.6));
    const double N3 = w3 * fmadd(w3, w3 - (0.9), (0.3 + 0.3 * 0.3)), D3 = fmadd(w3, (0.4), (0.3 * 0.3));
    g[0] = N1 * (D2 * D3);
    g[1] = N2 * (D1 * D3);
    g[2] = N3 * (D1 * D2);
    return (g[0] + g[1]) + g[2];
}

// L6, R6: six times the left-biased value at j+1/2 and the right-biased value at j-1/2
// of the cell with q = (m2, m1, c0, p1, p2).  eps4 = 4 eps: the sums S_k are four times
// eps + beta_k, a scale that cancels in the weights.  WW selects them: CNS_WENO_JS,
// Jiang-Shu alpha_k = c_k / S_k^2; CNS_WENO_Z, the WENO-Z weights of Borges et al. (2008),
// alpha_k = c_k (1 + (tau5/S_k)^2), tau5 = |S_1 - S_3|; CNS_WENO_M, the mapped weights
// above.  The alpha are scaled by S_1^2 S_2^2 S_3^2, so a normalisation takes one
// reciprocal.  Range, with S about the square of a jump of the scalar: the two Jiang-Shu
// sides share one, 1/D_L = D_R / (D_L D_R), a product of eight S factors (jumps to about
// 1e18); WENO-Z has products of six S factors for each side (1e25) and the mapped weights
// of four (1e37), so these take a reciprocal for each side.  From below the eps a plan
// admits bounds every S.
template <int WW>
__device__ __forceinline__ void weno5_cell6(double m2, double m1, double c0, double p1, double p2, double eps4,
                                            double &L6, double &R6) {
#pragma clang fp contract(off)
    const double k = 13.0 / 3.0;
    const double g0 = m1 - m2, g1 = c0 - m1, g2 = p1 - c0, g3 = p2 - p1;
    // second differences centred at j-1, j, j+1; one-sided and central first differences
    const double D1 = g1 - g0, D2 = g2 - g1, D3 = g3 - g2;
    const double e1 = fmadd(3.0, g1, -g0), e2 = g1 + g2, e3 = fmadd(3.0, g2, -g3);
    const double S1 = fmadd(e1, e1, fmadd(k * D1, D1, eps4)), S2 = fmadd(e2, e2, fmadd(k * D2, D2, eps4)),
            S3 = fmadd(e3, e3, fmadd(k * D3, D3, eps4));
    // candidates minus 6 q_j: at j+1/2 5 g1 - 2 g0, g1 + 2 g2, 4 g2 - g3; at j-1/2 minus
    // 4 g1 - g0, 2 g1 + g2, 5 g2 - 2 g3
    const double l1 = fmadd(2.0, e1, -g1), l2 = fmadd(2.0, g2, g1), l3 = e3 + g2;
    const double r1 = e1 + g1, r2 = fmadd(2.0, g1, g2), r3 = fmadd(2.0, e3, -g2);
    const double d1 = S1 * S1, d2 = S2 * S2, d3 = S3 * S3;
    double a1 = d2 * d3, a2 = d1 * d3, a3 = d1 * d2;
    if constexpr (WW == CNS_WENO_Z) {
        const double t = S1 - S3, tt = t * t;
        a1 = (d1 + tt) * a1, a2 = (d2 + tt) * a2, a3 = (d3 + tt) * a3;
    }
    const double t2 = 6.0 * a2, s = (a1 + a3) + t2;
    const double dL = fmadd(2.0, a3, s), dR = fmadd(2.0, a1, s);  // a1 + 6 a2 + 3 a3, 3 a1 + 6 a2 + a3
    const double b1 = 3.0 * a1, b3 = 3.0 * a3;
    double xL, xR;
    if constexpr (WW == CNS_WENO_M) {
        const double iL = rcp(dL), iR = rcp(dR);
        double gL[3], gR[3];
        const double GL = weno_map(a1 * iL, t2 * iL, b3 * iL, gL), GR = weno_map(a3 * iR, t2 * iR, b1 * iR, gR);
        const double q = rcp(GL * GR);
        xL = fmadd(gL[0], l1, fmadd(gL[1], l2, gL[2] * l3)) * (GR * q);
        xR = fmadd(gR[0], r3, fmadd(gR[1], r2, gR[2] * r1)) * (GL * q);
    } else {
        const double nL = fmadd(a1, l1, fmadd(t2, l2, b3 * l3)), nR = fmadd(a3, r3, fmadd(t2, r2, b1 * r1));
        if constexpr (WW == CNS_WENO_JS) {
            const double r = rcp(dL * dR);
            xL = nL * (dR * r);
            xR = nR * (dL * r);
        } else {
            xL = nL * rcp(dL);
            xR = nR * rcp(dR);
        }
    }
    L6 = fmadd(6.0, c0, xL);
    R6 = fmadd(6.0, c0, -xR);
}

// ---------------------------------------------------------------------------
// Sec. 2.1: convective flux along DIR of the conserved state w[5], components 1-4 (the
// density's flux is the momentum w[1 + DIR] itself)
// ---------------------------------------------------------------------------
template <typename T, int DIR>
__device__ __forceinline__ void euler_flux(const T w[5], T gm1, T f[4]) {
#pragma clang fp contract(off)
    const T inv = rcp(w[0]);
    const T vx = w[1] * inv, vy = w[2] * inv, vz = w[3] * inv;
    const T p = gm1 * fmadd(T(-0.5), fmadd(w[1], vx, fmadd(w[2], vy, w[3] * vz)), w[4]);
    const T vn = DIR == 0 ? vx : (DIR == 1 ? vy : vz);
    f[0] = DIR == 0 ? fmadd(w[1], vn, p) : w[1] * vn;
    f[1] = DIR == 1 ? fmadd(w[2], vn, p) : w[2] * vn;
    f[2] = DIR == 2 ? fmadd(w[3], vn, p) : w[3] * vn;
    f[3] = (w[4] + p) * vn;
}

// What the Roe average takes from a cell: sqrt(rho), velocity, total enthalpy.
template <typename T>
struct RoeCell {
    T s, v[3], H;
};
template <typename T>
__device__ __forceinline__ RoeCell<T> roe_cell(const T w[5], T gm1) {
#pragma clang fp contract(off)
    RoeCell<T> c;
    const T r = rsq(w[0]), i = r * r;  // 1/sqrt(rho) gives both sqrt(rho) = rho / sqrt(rho) and 1/rho
    c.s = w[0] * r;
#pragma unroll
    for (int d = 0; d < 3; ++d) c.v[d] = w[1 + d] * i;
    const T p = gm1 * fmadd(T(-0.5), fmadd(w[1], c.v[0], fmadd(w[2], c.v[1], w[3] * c.v[2])), w[4]);
    c.H = (w[4] + p) * i;
    return c;
}

// The nine distinct scalars that are reconstructed along a line: the state (0-4) and the
// fluxes of momentum and energy (5-8); the mass flux is the momentum along the line, so
// its reconstructions are those of that state component.
constexpr int kNS = 9;

// ---------------------------------------------------------------------------
// Sec. 2.2: interface flux H = (f^L + f^R)/2 - |A| (u^R - u^L)/2 between the cells a
// (= u_j) and b (= u_{j+1}) from the jumps du = u^R - u^L and the sums Fs = f^L + f^R of
// the six-fold reconstructions: |A| at the Roe average with Harten's fix on every
// eigenvalue, by wave strengths.  The dissipation is linear in the jump, so H = (6 F -
// 6 D) / 12.
// ---------------------------------------------------------------------------
template <typename T, int DIR>
__device__ __forceinline__ void interface_flux(const T du[5], const T Fs[5], const RoeCell<T> &a, const RoeCell<T> &b,
                                               T gm1, T delta, T Hf[5]) {
#pragma clang fp contract(off)
    constexpr int N = DIR, T1 = (DIR + 1) % 3, T2 = (DIR + 2) % 3;
    T v[3], D[5];
    const T iw = rcp(a.s + b.s);
    const T wa = a.s * iw, wb = b.s * iw;
#pragma unroll
    for (int d = 0; d < 3; ++d) v[d] = fmadd(wa, a.v[d], wb * b.v[d]);
    const T H = fmadd(wa, a.H, wb * b.H);
    const T hq2 = T(0.5) * fmadd(v[0], v[0], fmadd(v[1], v[1], v[2] * v[2]));
    const T c2 = gm1 * (H - hq2);
    const T ic = rsq(c2);
    const T c = c2 * ic;
    const T vn = v[N];

    // wave strengths alpha = X^-1 du
    const T at1 = fmadd(-v[T1], du[0], du[1 + T1]);
    const T at2 = fmadd(-v[T2], du[0], du[1 + T2]);
    const T dEb = fmadd(-at1, v[T1], fmadd(-at2, v[T2], du[4]));
    const T a2 = gm1 * (ic * ic) * fmadd(du[0], fmadd(-vn, vn, H), fmadd(vn, du[1 + N], -dEb));
    const T a1 = fmadd(-c, a2, fmadd(du[0], vn + c, -du[1 + N])) * (T(0.5) * ic);
    const T a5 = du[0] - (a1 + a2);

    const T hd = T(0.5) / delta;  // loop invariant
    const T l1 = harten_abs(vn - c, delta, hd), l2 = harten_abs(vn, delta, hd), l5 = harten_abs(vn + c, delta, hd);
    const T s1 = l1 * a1, s2 = l2 * a2, s5 = l5 * a5, st1 = l2 * at1, st2 = l2 * at2;

    // D = sum_k |lam_k| alpha_k K_k with the right eigenvectors K_k
    const T ssum = (s1 + s2) + s5, cd = c * (s5 - s1);
    D[0] = ssum;
    D[1 + N] = fmadd(ssum, v[N], cd);
    D[1 + T1] = fmadd(ssum, v[T1], st1);
    D[1 + T2] = fmadd(ssum, v[T2], st2);
    // s1 (H - vn c) + s2 q2/2 + s5 (H + vn c) + st1 v_t1 + st2 v_t2
    D[4] = fmadd(s1 + s5, H, fmadd(vn, cd, fmadd(s2, hq2, fmadd(st1, v[T1], st2 * v[T2]))));
#pragma unroll
    for (int k = 0; k < 5; ++k) Hf[k] = (Fs[k] - D[k]) * (T(1) / T(12));
}

// The jump and flux sum of component v from the face values of scalar c on the two sides
// (0-4 the state, 5-8 the fluxes of components 1-4)
template <typename T, int DIR>
__device__ __forceinline__ void face_pair(int c, T l, T r, T du[5], T Fs[5]) {
    if (c < 5) {
        du[c] = r - l;
        if (c == 1 + DIR) Fs[0] = l + r;
    } else {
        Fs[c - 4] = l + r;
    }
}

// 5-point 4th-order central first derivative (times h)
template <typename T>
__device__ __forceinline__ T dcen(T m2, T m1, T p1, T p2) {
    return (T(8) * (p1 - m1) - (p2 - m2)) * (T(1) / T(12));
}

}  // namespace cns
