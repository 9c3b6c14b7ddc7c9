// cns_device_adj.h -- hand-written reverse-mode (vector-Jacobian) products of the
// device arithmetic in cns_device.h, FP64.  Each *_vjp function recomputes the
// forward values it needs and ADDS the input adjoints to its outputs (weno5_cell_vjp and
// roe_mean_vjp set them).
#pragma once
#include "cns_device.h"

namespace cns {

// d|lam|_H / d lam of Harten's fix (0 at lam = 0 when delta = 0); idelta = 1/delta.
// Written with selects, no branches.
__device__ __forceinline__ double harten_dabs(double lam, double delta, double idelta) {
    const double sgn = lam > 0.0 ? 1.0 : (lam < 0.0 ? -1.0 : 0.0);
    return fabs(lam) >= delta ? sgn : lam * idelta;
}

// ---------------------------------------------------------------------------
// One biased reconstruction V = sum_k w_k q_k from the plain candidates q_k and the
// smoothness sums s_k = eps + beta_k: the value, the final weights w_k and dV/dbeta_k.
// With w_k = alpha_k / A and A = sum alpha:  dV/dbeta_j = sum_k (q_k - V) dalpha_k/dbeta_j / A.
//   JS: alpha_k = c_k / s_k^2, so dV/dbeta_j = -2 (q_j - V) w_j / s_j; the weights in
//       product form, t_k = prod_{i != k} s_i, P = s1 s2 s3, a_k = c_k t_k^2,
//       w_k = a_k P iPA and w_k / s_k = a_k t_k iPA with iPA = 1 / (P sum a).
//   Z:  alpha_k = c_k + tau z_k with z_k = c_k tau / s_k^2, tau = |beta1 - beta3|:
//       dV/dbeta_j = (1/A) [-2 (q_j - V) tau z_j / s_j + dtau/dbeta_j 2 sum_k (q_k - V) z_k].
//   M:  the JS weights u_k mapped, g_k = c_k + (u_k - c_k)^3 / D_k, D_k = c_k^2 + u_k (1 - 2 c_k),
//       w_k = g_k / G; with gamma_k = (q_k - V) g'_k / G,
//       dV/dbeta_j = -2 (u_j / s_j) (gamma_j - sum_k gamma_k u_k).
// ---------------------------------------------------------------------------
template <int WW>
__device__ __forceinline__ void weno_side_vjp(double s1, double s2, double s3, double q1, double q2, double q3,
                                              double &V, double w[3], double dV[3]) {
    if constexpr (WW == CNS_WENO_Z) {
        const double tau = fabs(s1 - s3);
        const double i1 = rcp(s1), i2 = rcp(s2), i3 = rcp(s3);
        const double z1 = 0.1 * tau * (i1 * i1), z2 = 0.6 * tau * (i2 * i2), z3 = 0.3 * tau * (i3 * i3);
        const double a1 = 0.1 + tau * z1, a2 = 0.6 + tau * z2, a3 = 0.3 + tau * z3;
        const double iA = rcp(a1 + a2 + a3);
        w[0] = a1 * iA, w[1] = a2 * iA, w[2] = a3 * iA;
        V = w[0] * q1 + w[1] * q2 + w[2] * q3;
        const double sg = s1 > s3 ? 1.0 : (s1 < s3 ? -1.0 : 0.0);
        const double P = 2.0 * ((q1 - V) * z1 + (q2 - V) * z2 + (q3 - V) * z3);
        dV[0] = iA * (-2.0 * (q1 - V) * tau * z1 * i1 + sg * P);
        dV[1] = iA * (-2.0 * (q2 - V) * tau * z2 * i2);
        dV[2] = iA * (-2.0 * (q3 - V) * tau * z3 * i3 - sg * P);
    } else {
        const double t1 = s2 * s3, t2 = s1 * s3, t3 = s1 * s2;
        const double a1 = 0.1 * (t1 * t1), a2 = 0.6 * (t2 * t2), a3 = 0.3 * (t3 * t3);
        const double iPA = rcp((t3 * s3) * (a1 + a2 + a3));
        const double iA = (t3 * s3) * iPA;
        const double u1 = a1 * iA, u2 = a2 * iA, u3 = a3 * iA;                     // Jiang-Shu weights
        const double r1 = a1 * t1 * iPA, r2 = a2 * t2 * iPA, r3 = a3 * t3 * iPA;  // u_k / s_k
        if constexpr (WW == CNS_WENO_JS) {
            w[0] = u1, w[1] = u2, w[2] = u3;
            V = u1 * q1 + u2 * q2 + u3 * q3;
            dV[0] = -2.0 * (q1 - V) * r1;
            dV[1] = -2.0 * (q2 - V) * r2;
            dV[2] = -2.0 * (q3 - V) * r3;
        } else {
            static_assert(WW == CNS_WENO_M, "unknown WENO weights");
            const double c[3] = {0.1, 0.6, 0.3}, u[3] = {u1, u2, u3}, r[3] = {r1, r2, r3}, q[3] = {q1, q2, q3};
            double g[3], gp[3], G = 0.0;
#pragma unroll
            for (int k = 0; k < 3; ++k) {
                const double e = u[k] - c[k], D = c[k] * c[k] + u[k] * (1.0 - 2.0 * c[k]), iD = rcp(D);
                g[k] = c[k] + e * e * e * iD;
                gp[k] = e * e * (3.0 * D - e * (1.0 - 2.0 * c[k])) * (iD * iD);
                G += g[k];
            }
            const double iG = rcp(G);
            V = 0.0;
#pragma unroll
            for (int k = 0; k < 3; ++k) {
                w[k] = g[k] * iG;
                V += w[k] * q[k];
            }
            double gam[3], S = 0.0;
#pragma unroll
            for (int k = 0; k < 3; ++k) {
                gam[k] = (q[k] - V) * gp[k] * iG;
                S += gam[k] * u[k];
            }
#pragma unroll
            for (int k = 0; k < 3; ++k) dV[k] = -2.0 * r[k] * (gam[k] - S);
        }
    }
}

// ---------------------------------------------------------------------------
// The reconstructions of one cell transposed (weno5_cell6 with the weights WW): given the
// adjoints Lb6, Rb6 of L6 and R6, six times the left-biased value at the cell's right face and
// the right-biased value at its left face, SET qb[0..4] to dL6/dq^T Lb6 + dR6/dq^T Rb6 (q = j-2
// .. j+2); the values themselves are returned in L6, R6.
//
// As in the forward, the two values share the indicator sums S_k = 4 (eps + beta_k), and
// both are q_j plus a combination of differences.  With the candidates l_k (L) and -r_k (R)
// less 6 q_j, A_k = t_k^2, t_k the product of the other two S, and P = S1 S2 S3, the
// Jiang-Shu weights are (A1, 6 A2, 3 A3) / D_L and (3 A1, 6 A2, A3) / D_R, and an indicator
// sum receives from both sides at once: d(value)/dS_k = -2 w_k (candidate_k - value) / S_k
// with 1 / S_k = t_k / P.  About 120 FP64 operations for the two values of a cell (166 for
// the two values at an interface, whose sides have indicators of their own).
// ---------------------------------------------------------------------------
template <int WW>
__device__ __forceinline__ void weno5_cell_vjp(const double q[5], double eps4, double Lb6, double Rb6, double qb[5],
                                               double &L6, double &R6) {
    const double c0 = q[2];
    const double g0 = q[1] - q[0], g1 = c0 - q[1], g2 = q[3] - c0, g3 = q[4] - q[3];
    const double D1 = g1 - g0, D2 = g2 - g1, D3 = g3 - g2;
    const double e1 = 3.0 * g1 - g0, e2 = g1 + g2, e3 = 3.0 * g2 - g3;
    const double k = 13.0 / 3.0;
    const double k1 = k * D1, k2 = k * D2, k3 = k * D3;
    const double S1 = (k1 * D1 + eps4) + e1 * e1, S2 = (k2 * D2 + eps4) + e2 * e2, S3 = (k3 * D3 + eps4) + e3 * e3;
    const double l1 = 2.0 * e1 - g1, l2 = 2.0 * g2 + g1, l3 = e3 + g2;
    const double r1 = e1 + g1, r2 = 2.0 * g1 + g2, r3 = 2.0 * e3 - g2;
    double xL, xR;        // six times the values less 6 q_j (R: with the opposite sign)
    double lb[3], rb[3];  // adjoints of l_k, r_k
    double s1, s2, s3;    // twice the adjoints of S_k
    if constexpr (WW == CNS_WENO_JS) {
        const double t1 = S2 * S3, t2 = S1 * S3, t3 = S1 * S2;
        const double A1 = t1 * t1, A2 = t2 * t2, A3 = t3 * t3;
        const double B1 = 3.0 * A1, B2 = 6.0 * A2, B3 = 3.0 * A3;
        const double s = (A1 + A3) + B2;
        const double dL = 2.0 * A3 + s, dR = 2.0 * A1 + s;
        // 1/P shares the left side's reciprocal (seven S factors), not the two sides one (eight)
        const double P = t1 * S1, r = rcp(dL * P), iL = P * r, iR = rcp(dR);
        const double iP4 = -4.0 * (dL * r);
        xL = (A1 * l1 + (B2 * l2 + B3 * l3)) * iL;
        xR = (A3 * r3 + (B2 * r2 + B1 * r1)) * iR;
        const double hL = Lb6 * iL, hR = -Rb6 * iR;
        lb[0] = hL * A1, lb[1] = hL * B2, lb[2] = hL * B3;
        rb[0] = hR * B1, rb[1] = hR * B2, rb[2] = hR * A3;
        s1 = (iP4 * t1) * (lb[0] * (l1 - xL) + rb[0] * (r1 - xR));
        s2 = (iP4 * t2) * (lb[1] * (l2 - xL) + rb[1] * (r2 - xR));
        s3 = (iP4 * t3) * (lb[2] * (l3 - xL) + rb[2] * (r3 - xR));
    } else {
        double w[3], v[3], dl[3], dr[3];
        weno_side_vjp<WW>(S1, S2, S3, l1, l2, l3, xL, w, dl);
        weno_side_vjp<WW>(S3, S2, S1, r3, r2, r1, xR, v, dr);  // mirrored stencils
        lb[0] = Lb6 * w[0], lb[1] = Lb6 * w[1], lb[2] = Lb6 * w[2];
        rb[0] = -Rb6 * v[2], rb[1] = -Rb6 * v[1], rb[2] = -Rb6 * v[0];
        s1 = 2.0 * (Lb6 * dl[0] - Rb6 * dr[2]);
        s2 = 2.0 * (Lb6 * dl[1] - Rb6 * dr[1]);
        s3 = 2.0 * (Lb6 * dl[2] - Rb6 * dr[0]);
    }
    L6 = 6.0 * c0 + xL;
    R6 = 6.0 * c0 - xR;
    // S = 4 eps + (13/3) D^2 + e^2; candidates; differences
    const double d1 = k1 * s1, d2 = k2 * s2, d3 = k3 * s3;
    const double f1 = e1 * s1 + (2.0 * lb[0] + rb[0]), f2 = e2 * s2, f3 = e3 * s3 + (2.0 * rb[2] + lb[2]);
    const double h0 = -f1 - d1;
    const double h1 = (3.0 * f1 + f2) + (d1 - d2) + ((lb[1] - lb[0]) + (2.0 * rb[1] + rb[0]));
    const double h2 = (3.0 * f3 + f2) + (d2 - d3) + ((rb[1] - rb[2]) + (2.0 * lb[1] + lb[2]));
    const double h3 = d3 - f3;
    qb[0] = -h0;
    qb[1] = h0 - h1;
    qb[2] = 6.0 * (Lb6 + Rb6) + (h1 - h2);
    qb[3] = h2 - h3;
    qb[4] = h3;
}

// wb += (df/dw)^T fb for the convective flux along DIR (the Euler flux Jacobian).
// With v = m / rho, K = |v|^2 / 2, p = (gamma-1)(e - rho K), H = (e + p) / rho,
// phi = fb[1..3], psi = fb[4] and s = (gamma-1)(phi_n + psi v_n):
//   rho:  s K - v_n (phi.v + psi H)
//   m_j:  v_n phi_j - s v_j, plus fb[0] + phi.v + psi H for j = n
//   e:    s + psi v_n
template <int DIR>
__device__ __forceinline__ void euler_flux_vjp(const double w[5], double gm1, const double fb[5], double wb[5]) {
    const double inv = rcp(w[0]);
    const double v[3] = {w[1] * inv, w[2] * inv, w[3] * inv};
    const double K = 0.5 * (v[0] * v[0] + v[1] * v[1] + v[2] * v[2]);
    const double p = gm1 * (w[4] - w[0] * K);
    const double H = (w[4] + p) * inv;
    const double vn = v[DIR];
    const double s = gm1 * (fb[1 + DIR] + fb[4] * vn);
    const double dotH = fb[1] * v[0] + fb[2] * v[1] + fb[3] * v[2] + fb[4] * H;
    wb[0] += s * K - vn * dotH;
#pragma unroll
    for (int j = 0; j < 3; ++j) wb[1 + j] += vn * fb[1 + j] - s * v[j] + (j == DIR ? fb[0] + dotH : 0.0);
    wb[4] += s + fb[4] * vn;
}

// ---------------------------------------------------------------------------
// Roe dissipation (wave-strength form) D = M(a, b) du: linear in the jump du, with M from
// the Roe average of the cell states a, b alone (Harten's fix acts on the eigenvalues).
// Given Db, the transpose product in three parts, so that little is held at a time:
//   roe_jump_vjp:  dub += M^T Db (needs no du);
//   roe_mean_vjp:  the adjoints of the Roe-averaged velocity and enthalpy (needs du);
//   roe_cells_vjp: from these ab, bb += the adjoints of the states; what it needs of the
//     cells is formed from the states and pressures again.
// ---------------------------------------------------------------------------
// The Roe average of the states a, b (pressures pa, pb) and the fixed eigenvalues; ra, rb =
// 1/sqrt(rho), wa, wb the weights and iw = 1 / (sqrt(rho_a) + sqrt(rho_b)).
struct RoeFace {
    double ra, rb, iw, wa, wb, v[3], H, q2, c, ic, ic2, l1, l2, l5;
};
template <int DIR>
__device__ __forceinline__ RoeFace roe_face(const double a[5], double pa, const double b[5], double pb, double gm1,
                                            double delta) {
    RoeFace R;
    R.ra = rsq(a[0]), R.rb = rsq(b[0]);
    R.iw = rcp(a[0] * R.ra + b[0] * R.rb);
    // wa va = (a_k / sqrt(rho_a)) iw
    const double xa = R.ra * R.iw, xb = R.rb * R.iw;
    R.wa = a[0] * xa, R.wb = b[0] * xb;
#pragma unroll
    for (int k = 0; k < 3; ++k) R.v[k] = xa * a[1 + k] + xb * b[1 + k];
    R.H = xa * (a[4] + pa) + xb * (b[4] + pb);
    R.q2 = R.v[0] * R.v[0] + R.v[1] * R.v[1] + R.v[2] * R.v[2];
    const double c2 = gm1 * (R.H - 0.5 * R.q2);
    R.ic = rsq(c2);
    R.c = c2 * R.ic, R.ic2 = R.ic * R.ic;
    const double vn = R.v[DIR], hd = 0.5 / delta;
    R.l1 = harten_abs(vn - R.c, delta, hd), R.l2 = harten_abs(vn, delta, hd), R.l5 = harten_abs(vn + R.c, delta, hd);
    return R;
}

// The reverse of the wave strengths common to both products: the adjoints of alpha and
// lambda alpha, down to X's.
struct RoeStrengths {
    double a1b, a2b, a5b, at1b, at2b, numb, Xb;
    double s1b, s2b, s5b, st1b, st2b;
};
template <int DIR>
__device__ __forceinline__ RoeStrengths roe_strengths_vjp(const RoeFace &R, double gm1, const double Db[5]) {
    constexpr int N = DIR, T1 = (DIR + 1) % 3, T2 = (DIR + 2) % 3;
    const double vnc = R.v[N] * R.c;
    RoeStrengths r;
    // D0 = ssum, D[1+k] = ssum v_k + ..., D4 = s1 (H - vn c) + s2 q2/2 + s5 (H + vn c) + st1 v_t1
    // + st2 v_t2; D[1+T] += st, D[1+N] += c (s5 - s1)
    const double ssumb = Db[0] + Db[1] * R.v[0] + Db[2] * R.v[1] + Db[3] * R.v[2];
    r.s1b = Db[4] * (R.H - vnc) - Db[1 + N] * R.c + ssumb;
    r.s5b = Db[4] * (R.H + vnc) + Db[1 + N] * R.c + ssumb;
    r.s2b = Db[4] * 0.5 * R.q2 + ssumb;
    r.st1b = Db[4] * R.v[T1] + Db[1 + T1];
    r.st2b = Db[4] * R.v[T2] + Db[1 + T2];
    // s = |lam| alpha; a5 = du0 - (a1 + a2); a1 = num / (2c); num = du0 (vn + c) - du_n - c a2
    r.a5b = r.s5b * R.l5;
    r.a1b = r.s1b * R.l1 - r.a5b;
    r.numb = r.a1b * (0.5 * R.ic);
    r.a2b = r.s2b * R.l2 - r.a5b - r.numb * R.c;
    // a2 = gm1/c2 X;  X = du0 (H - vn^2) + vn du_n - dEb;  dEb = du4 - at1 v_t1 - at2 v_t2; at = du_t - v_t du0
    r.Xb = r.a2b * gm1 * R.ic2;
    r.at1b = r.st1b * R.l2 + r.Xb * R.v[T1];
    r.at2b = r.st2b * R.l2 + r.Xb * R.v[T2];
    return r;
}
template <int DIR>
__device__ __forceinline__ void roe_jump_vjp(const RoeFace &R, double gm1, const double Db[5], double dub[5]) {
    constexpr int N = DIR, T1 = (DIR + 1) % 3, T2 = (DIR + 2) % 3;
    const double vn = R.v[N];
    const RoeStrengths r = roe_strengths_vjp<DIR>(R, gm1, Db);
    dub[0] += r.a5b + r.numb * (vn + R.c) + r.Xb * (R.H - vn * vn) - r.at1b * R.v[T1] - r.at2b * R.v[T2];
    dub[1 + N] += r.Xb * vn - r.numb;
    dub[1 + T1] += r.at1b;
    dub[1 + T2] += r.at2b;
    dub[4] -= r.Xb;
}
template <int DIR>
__device__ __forceinline__ void roe_mean_vjp(const RoeFace &R, double gm1, double delta, const double du[5],
                                             const double Db[5], double vbar[3], double &Hbar) {
    constexpr int N = DIR, T1 = (DIR + 1) % 3, T2 = (DIR + 2) % 3;
    const double vn = R.v[N], c = R.c, idelta = 1.0 / delta;
    const RoeStrengths r = roe_strengths_vjp<DIR>(R, gm1, Db);
    // the wave strengths of du
    const double at1 = du[1 + T1] - R.v[T1] * du[0], at2 = du[1 + T2] - R.v[T2] * du[0];
    const double dEb = du[4] - at1 * R.v[T1] - at2 * R.v[T2];
    const double a2 = gm1 * R.ic2 * (du[0] * (R.H - vn * vn) + vn * du[1 + N] - dEb);
    const double a1 = (du[0] * (vn + c) - du[1 + N] - c * a2) * (0.5 * R.ic), a5 = du[0] - (a1 + a2);
    const double s1 = R.l1 * a1, s2 = R.l2 * a2, s5 = R.l5 * a5, ssum = s1 + s2 + s5, sd = s5 - s1;
    Hbar = Db[4] * (s1 + s5) + r.Xb * du[0];
    double vnb = Db[4] * sd * c, cb = Db[4] * sd * vn + Db[1 + N] * sd, q2b = Db[4] * 0.5 * s2;
    vbar[N] = Db[1 + N] * ssum;
    vbar[T1] = Db[4] * R.l2 * at1 + Db[1 + T1] * ssum + r.Xb * at1 - r.at1b * du[0];
    vbar[T2] = Db[4] * R.l2 * at2 + Db[1 + T2] * ssum + r.Xb * at2 - r.at2b * du[0];
    const double x1 = r.s1b * a1 * harten_dabs(vn - c, delta, idelta), x5 = r.s5b * a5 * harten_dabs(vn + c, delta, idelta);
    vnb += x1 + (r.s2b * a2 + r.st1b * at1 + r.st2b * at2) * harten_dabs(vn, delta, idelta) + x5;
    cb += x5 - x1;
    cb -= r.a1b * a1 * R.ic;
    vnb += r.numb * du[0];
    cb += r.numb * (du[0] - a2);
    vnb += r.Xb * (du[1 + N] - 2.0 * vn * du[0]);
    vbar[N] += vnb;
    // c = sqrt(c2); c2 = gm1 (H - q2/2); q2 = |v|^2
    const double c2b = cb * (0.5 * R.ic) - r.a2b * a2 * R.ic2;
    Hbar += c2b * gm1;
    q2b -= 0.5 * gm1 * c2b;
#pragma unroll
    for (int k = 0; k < 3; ++k) vbar[k] += 2.0 * R.v[k] * q2b;
}
// H = wa Ha + wb Hb, v = wa va + wb vb; wa = sa iw, wb = sb iw, iw = 1/(sa + sb), s = sqrt(rho);
// Ha = (a4 + pa) / a0, va = a_k / a0
__device__ __forceinline__ void roe_cells_vjp(const RoeFace &R, const double a[5], double pa, const double b[5],
                                              double pb, double gm1, const double vbar[3], double Hbar, double ab[5],
                                              double bb[5]) {
    const double ia = R.ra * R.ra, ib = R.rb * R.rb;
    const double Ha = (a[4] + pa) * ia, Hb = (b[4] + pb) * ib;
    const double wab = Hbar * Ha + (vbar[0] * a[1] + vbar[1] * a[2] + vbar[2] * a[3]) * ia;
    const double wbb = Hbar * Hb + (vbar[0] * b[1] + vbar[1] * b[2] + vbar[2] * b[3]) * ib;
    // sa' = wab iw - iw (wab wa + wbb wb), and d sqrt(rho)/d rho = 1/(2 sqrt(rho))
    const double t = wab * R.wa + wbb * R.wb;
    const double sab = (wab - t) * R.iw, sbb = (wbb - t) * R.iw;
    auto cell = [&](const double w[5], double H, double i, double wt, double s0, double out[5]) {
        const double Hw = Hbar * wt, p = Hw * i;  // adjoints of H of the cell, and of e + p
        const double q = -0.5 * gm1 * p;          // of m.v
        double is = Hw * H;                       // of 1/rho, times rho
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            const double vk = vbar[k] * wt + q * w[1 + k], v = w[1 + k] * i;
            out[1 + k] += q * v + vk * i;
            is += vk * v;
        }
        out[4] += p + gm1 * p;
        out[0] += s0 - is * i;
    };
    cell(a, Ha, ia, R.wa, sab * (0.5 * R.ra), ab);
    cell(b, Hb, ib, R.wb, sbb * (0.5 * R.rb), bb);
}

// Ends a stage: the compiler neither merges loads nor moves arithmetic across it, so that a
// stage's values are not all live at once.
__device__ __forceinline__ void adj_stage_fence() {
    asm volatile("" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
}

}  // namespace cns
