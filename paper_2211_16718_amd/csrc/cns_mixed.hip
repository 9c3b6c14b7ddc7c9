// cns_mixed.hip -- kernels of the mixed form: FP32 state and flux arithmetic, FP64
// smoothness-indicator sums and accumulator.
//
// The mixed form keeps the interface-by-interface evaluation (both biases at j+1/2 from
// the six points j-2 .. j+3) and the nine stored viscous fluxes.  In FP32 the rounding of
// every intermediate shows in the results: the cell-by-cell evaluation and the one-pass
// viscous terms of the FP64 kernels ran 1.3 x faster here as well (256^3 step 6.5 against
// 8.5 ms) and no further from the FP64 solution, but they move the diagnostics, which are
// FP64 numbers, by 4.5e-8 relative and single states by an ulp.
//
// One RHS: k_visc_flux (u -> G = (tau_xx, tau_yy, tau_zz, tau_xy, tau_xz, tau_yz, E_x, E_y,
// E_z), E_d = v.tau_d - q_d), the x sweep (u, G -> rhs), the y and z sweeps (accumulate; z
// with the Runge-Kutta update).  The viscous term along d enters through the interface flux
// (-G_{j-1} + 7 G_j + 7 G_{j+1} - G_{j+2}) / 12, whose difference is the 5-point central
// derivative of G.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "cns_batch.h"
#include "cns_mixed.h"

namespace cns {
namespace mixed {

// ---------------------------------------------------------------------------
// WENO5, left- and right-biased values at j+1/2 from q_{j-2} .. q_{j+3} (the two share two
// of their three candidates and two of their four second differences)
// ---------------------------------------------------------------------------
// Nonlinear weights of one reconstruction from its three indicators b1..b3 (in B) and
// candidates c1..c3 (any common scale of b and eps, and of the c, passes through).
// WW selects the weights: CNS_WENO_JS, Jiang-Shu alpha_k = c_k / s_k^2 with
// s_k = eps + b_k; CNS_WENO_Z, the WENO-Z weights of Borges et al. (2008),
// alpha_k = c_k (1 + (tau5/s_k)^2) with tau5 = |b1 - b3|; CNS_WENO_M, the mapped
// weights of Henrick et al. (2005), the Jiang-Shu weights w_k passed through
// g_k(w) = w (c_k + c_k^2 - 3 c_k w + w^2) / (c_k^2 + w (1 - 2 c_k)) and renormalised.
// The alpha are scaled by s_1^2 s_2^2 s_3^2, the mapped values by the product of the
// three denominators, so one reciprocal serves the three weights of each
// normalisation.  The Z and mapped weights are formed in B (FP64) and normalised
// before any narrowing.
template <typename T, typename B, int WW>
__device__ __forceinline__ T weno5_combine(B b1, B b2, B b3, T eps, T c1, T c2, T c3) {
    if constexpr (WW == CNS_WENO_JS) {
        // products of four (eps + beta) factors would leave the
        // FP32 range at jumps of about 3e4 in the reconstructed value.  The s_k are first
        // scaled by the power of two of the smallest (exact), which puts t_k in [0.5, inf),
        // and capped at 2^31: a stencil whose t is capped has a weight below 2^-62 of the
        // smoothest one's, where the cap changes its contribution by less than the FP32
        // rounding of the smooth candidates (unless a jump exceeds the neighbouring values
        // by 1e11).  Then every product lies in [2^-4, 2^127), and the weights are
        // normalised before they multiply the candidates.
        T s1 = eps + T(b1), s2 = eps + T(b2), s3 = eps + T(b3);
        const int e = -__builtin_amdgcn_frexp_expf(fminf(s1, fminf(s2, s3)));
        const T cap = T(2147483648.0);
        T t1 = fminf(__builtin_amdgcn_ldexpf(s1, e), cap), t2 = fminf(__builtin_amdgcn_ldexpf(s2, e), cap),
          t3 = fminf(__builtin_amdgcn_ldexpf(s3, e), cap);
        T d1 = t1 * t1, d2 = t2 * t2, d3 = t3 * t3;
        T a1 = d2 * d3, a2 = T(6) * (d1 * d3), a3 = T(3) * (d1 * d2);
        T ir = rcp(a1 + a2 + a3);
        return (a1 * ir) * c1 + (a2 * ir) * c2 + (a3 * ir) * c3;
    } else if constexpr (WW == CNS_WENO_Z) {
        const B e = B(eps);
        B t = fabs(b1 - b3);
        B t2 = t * t;
        B s1 = e + b1, s2 = e + b2, s3 = e + b3;
        B d1 = s1 * s1, d2 = s2 * s2, d3 = s3 * s3;
        B a1 = B(0.1) * (d1 + t2) * (d2 * d3), a2 = B(0.6) * (d2 + t2) * (d1 * d3), a3 = B(0.3) * (d3 + t2) * (d1 * d2);
        B ia = rcp(a1 + a2 + a3);
        return T(a1 * ia) * c1 + T(a2 * ia) * c2 + T(a3 * ia) * c3;
    } else {
        static_assert(WW == CNS_WENO_M, "unknown WENO weights");
        const B e = B(eps);
        B s1 = e + b1, s2 = e + b2, s3 = e + b3;
        B d1 = s1 * s1, d2 = s2 * s2, d3 = s3 * s3;
        B a1 = B(0.1) * (d2 * d3), a2 = B(0.6) * (d1 * d3), a3 = B(0.3) * (d1 * d2);
        B ia = rcp(a1 + a2 + a3);
        B w1 = a1 * ia, w2 = a2 * ia, w3 = a3 * ia;  // Jiang-Shu weights
        // g_k = N_k / D_k with c = 1/10, 6/10, 3/10
        B N1 = w1 * (B(0.1) + B(0.1) * B(0.1) - B(0.3) * w1 + w1 * w1), D1 = B(0.1) * B(0.1) + w1 * B(0.8);
        B N2 = w2 * (B(0.6) + B(0.6) * B(0.6) - B(1.8) * w2 + w2 * w2), D2 = B(0.6) * B(0.6) + w2 * B(-0.2);
        B N3 = w3 * (B(0.3) + B(0.3) * B(0.3) - B(0.9) * w3 + w3 * w3), D3 = B(0.3) * B(0.3) + w3 * B(0.4);
        B g1 = N1 * (D2 * D3), g2 = N2 * (D1 * D3), g3 = N3 * (D1 * D2);
        B ig = rcp(g1 + g2 + g3);
        return T(g1 * ig) * c1 + T(g2 * ig) * c2 + T(g3 * ig) * c3;
    }
}

// Six times the left- and right-biased values, from four times the Jiang-Shu
// indicators: with eps4 = 4 eps every alpha_k scales by the same 1/16, so the weights
// are those of the plain form; dropping the 1/6 of the candidates and the 13/12, 1/4 of
// the indicators saves a multiplication per candidate and per indicator.
template <typename T, typename B, int WW = CNS_WENO_JS>
__device__ __forceinline__ void weno5_lr6(T m2, T m1, T c0, T p1, T p2, T p3, T eps4, T &L6, T &R6) {
    // 4 x Jiang-Shu smoothness indicators, (13/3) D^2 + E^2, accumulated in B, from the
    // first differences g_i = q_{i+1} - q_i of the stencil (q = m2, m1, c0, p1, p2, p3):
    // the second differences D and the one-sided E are short combinations of them
    const B k = B(13) / B(3);
    const B bm2 = B(m2), bm1 = B(m1), bc0 = B(c0), bp1 = B(p1), bp2 = B(p2), bp3 = B(p3);
    const B g0 = bm1 - bm2, g1 = bc0 - bm1, g2 = bp1 - bc0, g3 = bp2 - bp1, g4 = bp3 - bp2;
    B da = g1 - g0;  // second differences centred at j-1, j, j+1, j+2
    B db = g2 - g1;
    B dc = g3 - g2;
    B dd = g4 - g3;
    // the one-sided terms only enter squared, so each is formed with whichever sign
    // keeps it one fused multiply-add
    B ea = B(3) * g1 - g0;  // m2 - 4 m1 + 3 c0
    B eb = g1 + g2;         // -(m1 - p1)
    B ec = B(3) * g2 - g3;  // -(3 c0 - 4 p1 + p2)
    B fa = B(3) * g3 - g4;  // -(p3 - 4 p2 + 3 p1)
    B fb = g2 + g3;         // p2 - c0
    B fc = B(3) * g2 - g1;  // 3 p1 - 4 c0 + m1
    // third-order candidates (times 6); the mirror reconstruction reuses L2 and L3
    T L1, L2, L3, R1;
    {
        L1 = T(2) * m2 - T(7) * m1 + T(11) * c0;
        L2 = -m1 + T(5) * c0 + T(2) * p1;
        L3 = T(2) * c0 + T(5) * p1 - p2;
        R1 = T(2) * p3 - T(7) * p2 + T(11) * p1;
    }
    {
        const B qb = k * db * db, qc = k * dc * dc;  // shared by the two biases
        B bL1 = k * da * da + ea * ea;
        B bL2 = qb + eb * eb;
        B bL3 = qc + ec * ec;
        B bR1 = k * dd * dd + fa * fa;
        B bR2 = qc + fb * fb;
        B bR3 = qb + fc * fc;
        L6 = weno5_combine<T, B, WW>(bL1, bL2, bL3, eps4, L1, L2, L3);
        R6 = weno5_combine<T, B, WW>(bR1, bR2, bR3, eps4, R1, L3, L2);
    }
}

// ---------------------------------------------------------------------------
// Sec. 2.1: convective flux along DIR of the conserved state w[5]
// ---------------------------------------------------------------------------
template <typename T, int DIR>
__device__ __forceinline__ void euler_flux5(const T w[5], T gm1, T f[5]) {
    T inv = rcp(w[0]);
    T vx = w[1] * inv, vy = w[2] * inv, vz = w[3] * inv;
    T p = gm1 * (w[4] - T(0.5) * (w[1] * vx + w[2] * vy + w[3] * vz));
    T vn = DIR == 0 ? vx : (DIR == 1 ? vy : vz);
    f[0] = w[1 + DIR];
    f[1] = w[1] * vn;
    f[2] = w[2] * vn;
    f[3] = w[3] * vn;
    f[1 + DIR] += p;
    f[4] = (w[4] + p) * vn;
}

// ---------------------------------------------------------------------------
// Sec. 2.2: Roe dissipation D = |A| (uR - uL) at the Roe average of the cell
// states a (= u_j) and b (= u_{j+1}), with Harten's fix on every eigenvalue.
// ---------------------------------------------------------------------------
template <typename T, int DIR>
__device__ __forceinline__ void roe_dissipation(const T a[5], const T b[5], const T du[5], T gamma, T delta,
                                                T D[5]) {
    constexpr int N = DIR, T1 = (DIR + 1) % 3, T2 = (DIR + 2) % 3;
    const T gm1 = gamma - T(1);
    // 1/sqrt(rho) gives both sqrt(rho) = rho / sqrt(rho) and 1/rho
    T ra = rsq(a[0]), rb = rsq(b[0]);
    T ia = ra * ra, ib = rb * rb;
    T va[3] = {a[1] * ia, a[2] * ia, a[3] * ia};
    T vb[3] = {b[1] * ib, b[2] * ib, b[3] * ib};
    T pa = gm1 * (a[4] - T(0.5) * (a[1] * va[0] + a[2] * va[1] + a[3] * va[2]));
    T pb = gm1 * (b[4] - T(0.5) * (b[1] * vb[0] + b[2] * vb[1] + b[3] * vb[2]));
    T Ha = (a[4] + pa) * ia, Hb = (b[4] + pb) * ib;
    T sa = a[0] * ra, sb = b[0] * rb;
    T iw = rcp(sa + sb);
    T wa = sa * iw, wb = sb * iw;
    T v[3] = {wa * va[0] + wb * vb[0], wa * va[1] + wb * vb[1], wa * va[2] + wb * vb[2]};
    T H = wa * Ha + wb * Hb;
    T q2 = v[0] * v[0] + v[1] * v[1] + v[2] * v[2];
    T c2 = gm1 * (H - T(0.5) * q2);
    T ic = rsq(c2);
    T c = c2 * ic;
    T vn = v[N];

    // wave strengths alpha = X^-1 du
    T at1 = du[1 + T1] - v[T1] * du[0];
    T at2 = du[1 + T2] - v[T2] * du[0];
    T dEb = du[4] - at1 * v[T1] - at2 * v[T2];
    T a2 = gm1 * (ic * ic) * (du[0] * (H - vn * vn) + vn * du[1 + N] - dEb);
    T a1 = (du[0] * (vn + c) - du[1 + N] - c * a2) * (T(0.5) * ic);
    T a5 = du[0] - (a1 + a2);

    const T hd = T(0.5) / delta;  // loop invariant
    // fused as the compiler chooses, as all of this file's arithmetic
    auto habs = [&](T lam) {
        const T a = fabs(lam);
        return (a >= delta) ? a : (lam * lam + delta * delta) * hd;
    };
    T l1 = habs(vn - c), l2 = habs(vn), l5 = habs(vn + c);
    T s1 = l1 * a1, s2 = l2 * a2, s5 = l5 * a5, st1 = l2 * at1, st2 = l2 * at2;

    // D = sum_k |lam_k| alpha_k K_k with the right eigenvectors K_k
    T ssum = s1 + s2 + s5;
    D[0] = ssum;
    D[1] = ssum * v[0];
    D[2] = ssum * v[1];
    D[3] = ssum * v[2];
    D[1 + N] += c * (s5 - s1);
    D[1 + T1] += st1;
    D[1 + T2] += st2;
    D[4] = s1 * (H - vn * c) + s2 * (T(0.5) * q2) + s5 * (H + vn * c) + st1 * v[T1] + st2 * v[T2];
}

// ----------------------------------------------------------------------------
// viscous fluxes
// ----------------------------------------------------------------------------
// primitives (u, v, w, T = gamma p / rho) of the state at linear index i
template <typename T>
__device__ __forceinline__ void prim_at(gptr<const T> u, size_t n3, size_t i, T gamma, T W[4]) {
#pragma clang fp contract(off)
    const T r = u[i], mx = u[n3 + i], my = u[2 * n3 + i], mz = u[3 * n3 + i], e = u[4 * n3 + i];
    const T inv = rcp(r);
    W[0] = mx * inv;
    W[1] = my * inv;
    W[2] = mz * inv;
    const T p = (gamma - T(1)) * (e - T(0.5) * (mx * W[0] + my * W[1] + mz * W[2]));
    W[3] = gamma * p * inv;
}

// The 5-point central difference (times h) rounded as written (no fused multiply-add):
// the viscous-flux kernel forms every value of G with contraction off, so that the
// variant that also accumulates the diagnostics (extra uses of the gradients) gives the
// same bits.
template <typename T>
__device__ __forceinline__ T dcen_nc(T m2, T m1, T p1, T p2) {
#pragma clang fp contract(off)
    return (T(8) * (p1 - m1) - (p2 - m2)) * (T(1) / T(12));
}

// Viscous fluxes at points: the 12 first derivatives of (u, v, w, T) by the 5-point
// central stencil, then tau, q and G.  A block owns a 32 x 8 (x, y) tile and marches
// along z over vsz planes.  Each thread keeps its own column's primitives at planes
// k-2 .. k+2 in registers (z derivatives); a thread that owns a point of the tile's halo
// ring keeps that point's primitives at planes k .. k+2 in its own LDS slots.  Plane k
// is staged in LDS from the two windows (x and y derivatives).  Each state value of a
// plane is loaded once per tile, and the column and the ring point of plane k+2 are
// loaded together, while the neighbouring tiles (same XCD, launched together) load the
// same lines for their own columns, so the halo comes from L2.
template <typename T>
__global__ __launch_bounds__(kPointThreads) void k_visc_flux(Launch L0) {
#pragma clang fp contract(off)
    const Launch L = with_params(L0);
    __shared__ T pl[4][kViscTY + 4][kViscTX + 4];
    __shared__ T rw[3][4][kViscRing];  // ring primitives, slot (plane - z0) mod 3
    int rhx, rhy;
    ring_pos(threadIdx.x, rhx, rhy);
    const bool ring = threadIdx.x < kViscRing;
    const int rt = ring ? threadIdx.x : 0;
    const VbRange R = vb_range(L.total);
    for (long long vb = R.vb; vb < R.end; vb += R.stride) {
        const int bi = find_box(L.off, L.nbox, vb);
        const BoxDesc &b = L.boxes[bi];
        const int nx = b.nx, ny = b.ny, nz = b.nz;
        const size_t n3 = b.n3, sz = (size_t)nx * ny;
        const long long lb = vb - L.off[bi];
        const int ntx = (nx + kViscTX - 1) / kViscTX, nty = (ny + kViscTY - 1) / kViscTY;
        const int x0 = (int)(lb % ntx) * kViscTX, y0 = (int)((lb / ntx) % nty) * kViscTY;
        const int vsz = b.vsz;
        const int z0 = (int)(lb / ((long long)ntx * nty)) * vsz, z1 = min(z0 + vsz, nz);
        const int tx = threadIdx.x % kViscTX, ty = threadIdx.x / kViscTX;
        const bool act = x0 + tx < nx && y0 + ty < ny;
        // a column past a ragged edge wraps periodically: its primitives are halo values
        // of the active columns beside it
        const size_t col = (size_t)wrapm(y0 + ty, ny) * nx + wrapm(x0 + tx, nx);
        const size_t rcol = (size_t)wrapm(y0 - 2 + rhy, ny) * nx + wrapm(x0 - 2 + rhx, nx);
        const gptr<const T> u = glob((const T *)state_ptr(b, L, L.in));
        const gptr<T> G = glob((T *)b.G);
        const T gamma = T(b.gamma);
        const T ihx = T(b.inv_h[0]), ihy = T(b.inv_h[1]), ihz = T(b.inv_h[2]);
        const T mu = T(b.mu), kcond = T(b.mu / ((b.gamma - 1.0) * b.prandtl));
        T Wz[5][4];  // this column's primitives at planes k-2 .. k+2
#pragma unroll
        for (int m = 0; m < 4; ++m) {
            const size_t ic = col + wrapi(z0 - 2 + m, nz) * sz;
            prim_at(u, n3, ic, gamma, Wz[m]);
        }
        if (ring) {
            for (int m = 0; m < 2; ++m) {
                T w4[4];
                prim_at(u, n3, rcol + wrapi(z0 + m, nz) * sz, gamma, w4);
#pragma unroll
                for (int c = 0; c < 4; ++c) rw[m][c][rt] = w4[c];
            }
        }
        int slot = 0;  // (k - z0) mod 3
        for (int k = z0; k < z1; ++k) {
            const int slot2 = slot == 0 ? 2 : slot - 1;  // (k + 2 - z0) mod 3
            prim_at(u, n3, col + wrapi(k + 2, nz) * sz, gamma, Wz[4]);
            if (ring) {
                T w4[4];
                prim_at(u, n3, rcol + wrapi(k + 2, nz) * sz, gamma, w4);
#pragma unroll
                for (int c = 0; c < 4; ++c) {
                    rw[slot2][c][rt] = w4[c];
                    pl[c][rhy][rhx] = rw[slot][c][rt];
                }
            }
#pragma unroll
            for (int c = 0; c < 4; ++c) pl[c][ty + 2][tx + 2] = Wz[2][c];
            __syncthreads();
            if (act) {
                T g[4][3];  // g[a][c] = d W_a / d x_c
#pragma unroll
                for (int a = 0; a < 4; ++a) {
                    g[a][0] = dcen_nc(pl[a][ty + 2][tx], pl[a][ty + 2][tx + 1], pl[a][ty + 2][tx + 3], pl[a][ty + 2][tx + 4]) * ihx;
                    g[a][1] = dcen_nc(pl[a][ty][tx + 2], pl[a][ty + 1][tx + 2], pl[a][ty + 3][tx + 2], pl[a][ty + 4][tx + 2]) * ihy;
                    g[a][2] = dcen_nc(Wz[0][a], Wz[1][a], Wz[3][a], Wz[4][a]) * ihz;
                }
                T div = g[0][0] + g[1][1] + g[2][2];
                T tdiv = T(2) / T(3) * div;
                T txx = mu * (T(2) * g[0][0] - tdiv);
                T tyy = mu * (T(2) * g[1][1] - tdiv);
                T tzz = mu * (T(2) * g[2][2] - tdiv);
                T txy = mu * (g[0][1] + g[1][0]);
                T txz = mu * (g[0][2] + g[2][0]);
                T tyz = mu * (g[1][2] + g[2][1]);
                const T vx = Wz[2][0], vy = Wz[2][1], vz = Wz[2][2];
                const size_t idx = (size_t)k * sz + col;
                // non-temporal stores: G is streamed to memory and read back by the sweeps
                // (at 128^3: 1.3 % faster step, at 512^3: 1.9 %)
                __builtin_nontemporal_store(txx, &G[idx]);
                __builtin_nontemporal_store(tyy, &G[n3 + idx]);
                __builtin_nontemporal_store(tzz, &G[2 * n3 + idx]);
                __builtin_nontemporal_store(txy, &G[3 * n3 + idx]);
                __builtin_nontemporal_store(txz, &G[4 * n3 + idx]);
                __builtin_nontemporal_store(tyz, &G[5 * n3 + idx]);
                __builtin_nontemporal_store(vx * txx + vy * txy + vz * txz + kcond * g[3][0], &G[6 * n3 + idx]);
                __builtin_nontemporal_store(vx * txy + vy * tyy + vz * tyz + kcond * g[3][1], &G[7 * n3 + idx]);
                __builtin_nontemporal_store(vx * txz + vy * tyz + vz * tzz + kcond * g[3][2], &G[8 * n3 + idx]);
            }
            __syncthreads();  // the next plane overwrites the LDS tile
#pragma unroll
            for (int m = 0; m < 4; ++m)
#pragma unroll
                for (int c = 0; c < 4; ++c) Wz[m][c] = Wz[m + 1][c];
            slot = slot == 2 ? 0 : slot + 1;
        }
    }
}

// which G field holds component (momentum x, y, z, energy) of the viscous flux along DIR
template <int DIR>
__device__ __forceinline__ constexpr int gcomp(int c) {
    return DIR == 0 ? (c == 0 ? 0 : c == 1 ? 3 : c == 2 ? 4 : 6)
                    : (DIR == 1 ? (c == 0 ? 3 : c == 1 ? 1 : c == 2 ? 5 : 7) : (c == 0 ? 4 : c == 1 ? 5 : c == 2 ? 2 : 8));
}

// A stage's sweeps run x, y, z.  The G field of component c along DIR is read for the
// last time in that stage by this sweep when no later sweep reads it (tau_xy: x then y;
// tau_xz: x then z; tau_yz: y then z); such loads, and the z sweep's loads of rhs and
// of the FP64 accumulator, are marked non-temporal so they do not displace lines that
// are read again.
template <int DIR, int C>
__device__ __forceinline__ constexpr bool g_last_read() {
    return DIR == 2 || (DIR == 1 && C != 2) || (DIR == 0 && (C == 0 || C == 3));
}
template <int DIR, int C, typename T>
__device__ __forceinline__ T load_g(gptr<const T> G, size_t n3, size_t o) {
    if constexpr (g_last_read<DIR, C>()) return __builtin_nontemporal_load(&G[gcomp<DIR>(C) * n3 + o]);
    else return G[gcomp<DIR>(C) * n3 + o];
}
// the same with the point's byte offset
template <int DIR, int C, typename T>
__device__ __forceinline__ T load_gb(gptr<const T> G, size_t n3, uint32_t bo) {
    if constexpr (g_last_read<DIR, C>()) return __builtin_nontemporal_load(elem(G, n3, gcomp<DIR>(C), bo));
    else return *elem(G, n3, gcomp<DIR>(C), bo);
}

// viscous term alone: out = sum_d D_d G_d (the viscous-only entry point)
template <typename T>
__global__ __launch_bounds__(kPointThreads) void k_visc_div(Launch L0) {
    const Launch L = with_params(L0);
    const VbRange R = vb_range(L.total);
    for (long long vb = R.vb; vb < R.end; vb += R.stride) {
        const int bi = find_box(L.off, L.nbox, vb);
        const BoxDesc &b = L.boxes[bi];
        const int nx = b.nx, ny = b.ny, nz = b.nz;
        const size_t n3 = b.n3;
        const size_t idx = (size_t)(vb - L.off[bi]) * kPointThreads + threadIdx.x;
        if (idx >= n3) continue;
        const gptr<const T> G = glob((const T *)b.G);
        const gptr<T> out = glob((T *)(L.out_ov ? L.out_ov : b.rhs));
        const T ihx = T(b.inv_h[0]), ihy = T(b.inv_h[1]), ihz = T(b.inv_h[2]);
        const int i = (int)(idx % nx);
        const int j = (int)((idx / nx) % ny);
        const int k = (int)(idx / ((size_t)nx * ny));
        const size_t sy = nx, sz = (size_t)nx * ny;
        const size_t row = idx - i, col = idx - j * sy, pil = idx - k * sz;
        const size_t x[4] = {row + wrapi(i - 2, nx), row + wrapi(i - 1, nx), row + wrapi(i + 1, nx),
                             row + wrapi(i + 2, nx)};
        const size_t y[4] = {col + wrapi(j - 2, ny) * sy, col + wrapi(j - 1, ny) * sy, col + wrapi(j + 1, ny) * sy,
                             col + wrapi(j + 2, ny) * sy};
        const size_t z[4] = {pil + wrapi(k - 2, nz) * sz, pil + wrapi(k - 1, nz) * sz, pil + wrapi(k + 1, nz) * sz,
                             pil + wrapi(k + 2, nz) * sz};
        out[idx] = T(0);
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            const gptr<const T> gx = G + gcomp<0>(c) * n3;
            const gptr<const T> gy = G + gcomp<1>(c) * n3;
            const gptr<const T> gz = G + gcomp<2>(c) * n3;
            T s = dcen(gx[x[0]], gx[x[1]], gx[x[2]], gx[x[3]]) * ihx;
            s += dcen(gy[y[0]], gy[y[1]], gy[y[2]], gy[y[3]]) * ihy;
            s += dcen(gz[z[0]], gz[z[1]], gz[z[2]], gz[z[3]]) * ihz;
            out[(1 + c) * n3 + idx] = s;
        }
    }
}

// ----------------------------------------------------------------------------
// convective sweeps
// ----------------------------------------------------------------------------
// Interface flux at j+1/2 from the states w and (VISC) the viscous fluxes g at j-1 .. j+2:
//   H = (f^L + f^R)/2 - |A| (u^R - u^L)/2 - (-g_{j-1} + 7 g_j + 7 g_{j+1} - g_{j+2})/12,
// from six-fold reconstructions, with the point fluxes read from the per-thread LDS ring of the
// marching sweep (slot sl[m] holds point j-2+m), one component at a time: the fence
// between components keeps the scheduler from hoisting all thirty LDS reads, which
// would hold them in registers across the whole reconstruction.
template <typename T, typename B, int DIR, bool VISC, int WW>
__device__ __forceinline__ void interface_flux_ring(const T w[6][5], const T *ring, const int sl[6], int bdim,
                                                    const T g[4][4], T gamma, T eps4, T delta, T H[5]) {
    T Fs[5], du[5], D[5];
#pragma unroll
    for (int v = 0; v < 5; ++v) {
        T fm[6];
#pragma unroll
        for (int m = 0; m < 6; ++m) fm[m] = ring[(sl[m] * 5 + v) * bdim];
        T FL, FR, UL, UR;
        weno5_lr6<T, B, WW>(fm[0], fm[1], fm[2], fm[3], fm[4], fm[5], eps4, FL, FR);
        weno5_lr6<T, B, WW>(w[0][v], w[1][v], w[2][v], w[3][v], w[4][v], w[5][v], eps4, UL, UR);
        Fs[v] = FL + FR;
        du[v] = UR - UL;
        __builtin_amdgcn_sched_barrier(0);
    }
    roe_dissipation<T, DIR>(w[2], w[3], du, gamma, delta, D);
#pragma unroll
    for (int v = 0; v < 5; ++v) H[v] = (Fs[v] - D[v]) * (T(1) / T(12));
    if constexpr (VISC) {
#pragma unroll
        for (int c = 0; c < 4; ++c)
            H[1 + c] -= (T(7) * (g[1][c] + g[2][c]) - (g[0][c] + g[3][c])) * (T(1) / T(12));
    }
}

// The same interface flux with every operand read from the rows kernel's LDS staging
// (component-major arrays of `per` points; q[m] is the position of point i-2+m), one
// component at a time behind a scheduling fence, so that the reconstruction holds
// only the operands of the component in flight.
template <typename T, typename B, int DIR, bool VISC, int WW>
__device__ __forceinline__ void interface_flux_lds(const T *su, const T *sf, const T *sg, int per, const int q[6],
                                                   T gamma, T eps4, T delta, T H[5]) {
    T Fs[5], du[5], D[5];
#pragma unroll
    for (int v = 0; v < 5; ++v) {
        const T *fv = sf + v * per, *uv = su + v * per;
        T FL, FR, UL, UR;
        weno5_lr6<T, B, WW>(fv[q[0]], fv[q[1]], fv[q[2]], fv[q[3]], fv[q[4]], fv[q[5]], eps4, FL, FR);
        weno5_lr6<T, B, WW>(uv[q[0]], uv[q[1]], uv[q[2]], uv[q[3]], uv[q[4]], uv[q[5]], eps4, UL, UR);
        Fs[v] = FL + FR;
        du[v] = UR - UL;
        __builtin_amdgcn_sched_barrier(0);
    }
    T a[5], b[5];
#pragma unroll
    for (int v = 0; v < 5; ++v) {
        a[v] = su[v * per + q[2]];
        b[v] = su[v * per + q[3]];
    }
    roe_dissipation<T, DIR>(a, b, du, gamma, delta, D);
#pragma unroll
    for (int v = 0; v < 5; ++v) H[v] = (Fs[v] - D[v]) * (T(1) / T(12));
    if constexpr (VISC) {
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            const T *gc = sg + c * per;
            H[1 + c] -= (T(7) * (gc[q[2]] + gc[q[3]]) - (gc[q[1]] + gc[q[4]])) * (T(1) / T(12));
        }
    }
}

enum { MODE_WRITE = 0, MODE_ACCUM = 1, MODE_RK = 2 };

// Lanes run over consecutive lines of the plane (coalesced).  For y, a block of W
// waves covers 64 lines times W consecutive segments, so neighbouring segments share
// their six-point halos in the CU's cache; for x and z a block covers 64 W lines of one
// segment (stacking z segments spreads a block over planes far apart in memory).
//
// The six point fluxes live in a per-thread ring in LDS (6 slots x 5 components,
// component-major across the wave so lanes hit distinct banks), read one component
// at a time; the registers this frees carry the loads of the next point and of the
// point's rhs, issued before the interface-flux arithmetic so their latency overlaps
// it (y sweep 12 % and fused-update sweep 6 % faster than a register window).  The
// fused update's u^n and accumulator are loaded ahead in the same way.
template <typename T, typename B, int DIR, int MODE, bool VISC, int WW>
__global__ __launch_bounds__(256, 2) void k_sweep(Launch L0) {
    const Launch L = with_params(L0);
    extern __shared__ unsigned char lds_raw[];
    // each wave's ring: slot s, component v of lane l at (s * 5 + v) * 64 + l, so the
    // component and slot strides are constants (immediate LDS offsets)
    constexpr int bdim = 64;
    T *ring = reinterpret_cast<T *>(lds_raw) + (threadIdx.x >> 6) * (30 * 64) + (threadIdx.x & 63);
    const VbRange R = vb_range(L.total);
    for (long long vb = R.vb; vb < R.end; vb += R.stride) {
        const int bi = find_box(L.off, L.nbox, vb);
        const BoxDesc &bx = L.boxes[bi];
        const SweepGeom sg = sweep_geom<DIR>(bx.nx, bx.ny, bx.nz);
        const int n = sg.nline;
        const int seg = bx.seg[DIR];
        const int nseg = (n + seg - 1) / seg;
        const long long lb = vb - L.off[bi];
        int pq, sgi;
        if constexpr (DIR == 1) {
            const int wpb = blockDim.x >> 6;
            const long long ncg = (sg.npq + 63) >> 6;
            pq = (int)((lb % ncg) << 6) + (int)(threadIdx.x & 63);
            sgi = (int)(lb / ncg) * wpb + (int)(threadIdx.x >> 6);
            if (pq >= sg.npq || sgi >= nseg) continue;
        } else {
            const size_t t = (size_t)lb * blockDim.x + threadIdx.x;
            if (t >= (size_t)sg.npq * nseg) continue;
            pq = (int)(t % sg.npq);
            sgi = (int)(t / sg.npq);
        }
        const int p = pq % sg.np, q = pq / sg.np;
        const size_t base = p * sg.pstride + q * sg.qstride;
        const int j0 = sgi * seg;
        const int j1 = min(j0 + seg, n);
        const size_t n3 = uni64(bx.n3);
        const gptr<const T> u = uni(glob((const T *)state_ptr(bx, L, L.in)));
        const gptr<const T> G = uni(glob((const T *)bx.G));
        const T gamma = T(bx.gamma), eps4 = T(4.0 * bx.eps), delta = T(bx.delta);
        const T gm1 = gamma - T(1);
        const T inv_dx = T(bx.inv_h[DIR]);
        const double dt = L.dt_ov > 0.0 ? L.dt_ov : bx.dt;
        // Every pointer the loop uses is read from the box table here, once: the loop
        // stores to global memory, which the compiler cannot tell apart from the table, so
        // a table read inside the loop would be repeated after every store, each time
        // behind a wait for all loads in flight (the ones issued ahead included).
        const gptr<const T> rhs_in = uni(glob((const T *)(MODE == MODE_RK ? bx.rhs : (L.out_ov ? L.out_ov : bx.rhs))));
        const gptr<const T> un = uni(glob((const T *)state_ptr(bx, L, BUF_U)));
        const gptr<double> acc = uni(glob(bx.acc));
        const gptr<T> unext = uni(glob((T *)state_ptr(bx, L, L.out)));
        const gptr<T> rhs_out = uni(glob((T *)(L.out_ov ? L.out_ov : bx.rhs)));

        T w[6][5], g[4][4], Hp[5], nw[5];
        // One step body computes everything, so every point flux and every interface
        // flux takes the same arithmetic in the same order wherever a segment starts:
        // results are bitwise independent of the segment length.  Step j takes point
        // j+3 (loaded one step ahead) and the viscous fluxes of point j+2; from j = j0-1
        // on it forms the interface flux at j+1/2 and from j = j0 on the flux difference
        // at point j.
        {
            const uint32_t bo = (uint32_t)((base + wrapi(j0 - 3, n) * sg.lstride) * sizeof(T));
#pragma unroll
            for (int v = 0; v < 5; ++v) nw[v] = *elem(u, n3, v, bo);
        }
        int snew = 3;  // ring slot of point j+3; point j-2+m sits in slot (snew + 1 + m) mod 6
        auto step = [&](const int j) {
#pragma unroll
            for (int m = 0; m < 5; ++m)
#pragma unroll
                for (int v = 0; v < 5; ++v) w[m][v] = w[m + 1][v];
#pragma unroll
            for (int v = 0; v < 5; ++v) w[5][v] = nw[v];
            // The window enters each step through an empty asm, so the two steps of a
            // pass share no arithmetic (the optimiser would otherwise form a point's Roe
            // terms once for both interfaces, outside the block where the other step
            // fuses them into multiply-adds): every interface flux is computed by the
            // same instructions in either step, bitwise as with one step per pass.
#pragma unroll
            for (int m = 0; m < 6; ++m)
#pragma unroll
                for (int v = 0; v < 5; ++v) asm volatile("" : "+v"(w[m][v]));
            {
                const uint32_t bo = (uint32_t)((base + wrapi(j + 4, n) * sg.lstride) * sizeof(T));
#pragma unroll
                for (int v = 0; v < 5; ++v) nw[v] = *elem(u, n3, v, bo);
            }
            if constexpr (VISC) {
#pragma unroll
                for (int m = 0; m < 3; ++m)
#pragma unroll
                    for (int c = 0; c < 4; ++c) g[m][c] = g[m + 1][c];
                const uint32_t bog = (uint32_t)((base + wrapi(j + 2, n) * sg.lstride) * sizeof(T));
                g[3][0] = load_gb<DIR, 0>(G, n3, bog);
                g[3][1] = load_gb<DIR, 1>(G, n3, bog);
                g[3][2] = load_gb<DIR, 2>(G, n3, bog);
                g[3][3] = load_gb<DIR, 3>(G, n3, bog);
#pragma unroll
                for (int m = 0; m < 3; ++m)
#pragma unroll
                    for (int c = 0; c < 4; ++c) asm volatile("" : "+v"(g[m][c]));
            }
            const int sold = snew;
            {
                T fn[5];
                euler_flux5<T, DIR>(w[5], gm1, fn);
#pragma unroll
                for (int v = 0; v < 5; ++v) ring[(snew * 5 + v) * bdim] = fn[v];
                snew = snew == 5 ? 0 : snew + 1;
            }
            if (j < j0 - 1) return;

            // output operands of point j, loaded before the interface-flux arithmetic
            const size_t o = base + (size_t)(j >= j0 ? j : j0) * sg.lstride;
            const uint32_t bo = (uint32_t)(o * sizeof(T)), boa = (uint32_t)(o * sizeof(double));
            T pr[5], pu[5];
            double pa[5];
            if (MODE != MODE_WRITE && j >= j0) {
#pragma unroll
                for (int v = 0; v < 5; ++v) {
                    if constexpr (MODE == MODE_RK) pr[v] = __builtin_nontemporal_load(elem(rhs_in, n3, v, bo));
                    else pr[v] = *elem(rhs_in, n3, v, bo);
                }
                if (MODE == MODE_RK && L.stage >= 2) {
                    // u^n: every later stage but the mixed form's RK4 stage 4, which
                    // needs only the accumulator
                    if (L.scheme == CNS_TVDRK3 || L.stage != 4) {
#pragma unroll
                        for (int v = 0; v < 5; ++v) pu[v] = *elem(un, n3, v, bo);
                    }
                    if (L.scheme != CNS_TVDRK3) {
#pragma unroll
                        for (int v = 0; v < 5; ++v) pa[v] = __builtin_nontemporal_load(elem(acc, n3, v, boa));
                    }
                }
            }

            T H[5];
            {
                int sl[6];
#pragma unroll
                for (int m = 0; m < 6; ++m) {
                    const int sm = sold + 1 + m;  // slot of point j-2+m (point j+3 is in sold)
                    sl[m] = sm >= 6 ? sm - 6 : sm;
                }
                interface_flux_ring<T, B, DIR, VISC, WW>(w, ring, sl, bdim, g, gamma, eps4, delta, H);
            }
            if (j >= j0) {
                if constexpr (MODE == MODE_RK) {
#pragma unroll
                    for (int v = 0; v < 5; ++v) {
                        const T r = -(H[v] - Hp[v]) * inv_dx;
                        const gptr<T> ue = elem(unext, n3, v, bo);
                        const gptr<double> ae = elem(acc, n3, v, boa);
                        const double k = double(pr[v] + r);
                        // w[2] holds the stage state at j: u^n itself in the first stage
                        const double us = double(w[2][v]);
                        if (L.scheme == CNS_TVDRK3) {
                            // Shu-Osher: U1 = u + dt k; U2 = 3/4 u + 1/4 (U1 + dt k);
                            // u^{n+1} = 1/3 u + 2/3 (U2 + dt k)
                            if (L.stage == 1) {
                                *ue = T(us + dt * k);
                            } else {
                                const double uo = double(pu[v]);
                                if (L.stage == 2) *ue = T(0.75 * uo + 0.25 * (us + dt * k));
                                else *ue = T((1.0 / 3.0) * uo + (2.0 / 3.0) * (us + dt * k));
                            }
                        } else if (L.stage == 1) {
                            *ae = us + (dt / 6.0) * k;
                            *ue = T(us + (0.5 * dt) * k);
                        } else if (L.stage == 2) {
                            const double uo = double(pu[v]);
                            *ae = pa[v] + (dt / 3.0) * k;
                            *ue = T(uo + (0.5 * dt) * k);
                        } else if (L.stage == 3) {
                            const double uo = double(pu[v]);
                            *ae = pa[v] + (dt / 3.0) * k;
                            *ue = T(uo + dt * k);
                        } else {
                            *ue = T(pa[v] + (dt / 6.0) * k);
                        }
                    }
                } else {
#pragma unroll
                    for (int v = 0; v < 5; ++v) {
                        const T r = -(H[v] - Hp[v]) * inv_dx;
                        if constexpr (MODE == MODE_WRITE) *elem(rhs_out, n3, v, bo) = r;
                        else *elem(rhs_out, n3, v, bo) = pr[v] + r;
                    }
                }
            }
#pragma unroll
            for (int v = 0; v < 5; ++v) Hp[v] = H[v];
        };
        // Two steps per pass: the window shifts of the first step become register
        // renamings instead of copies (y sweep 64 -> 26, z sweep 66 -> 30 64-bit moves
        // per point).
        int j = j0 - 6;
#pragma nounroll
        for (; j + 1 < j1; j += 2) {
            step(j);
            step(j + 1);
        }
        if (j < j1) step(j);
    }
}

// ----------------------------------------------------------------------------
// x sweep with whole periodic rows staged in LDS: one thread per point and per
// interface, lanes along x (coalesced loads and stores), `rows` rows per block of
// 256 threads, each thread handling up to P points.  Every interface of a row is
// computed once; the periodic wrap happens in LDS.
// ----------------------------------------------------------------------------
template <typename T, typename B, bool VISC, int P, int WW>
__global__ __launch_bounds__(kRowThreads, 2) void k_sweep_x_rows(Launch L0) {
    const Launch L = with_params(L0);
    extern __shared__ unsigned char lds_raw[];
    T *lds = reinterpret_cast<T *>(lds_raw);
    // A block walks over several row groups (grid stride).  With one point per thread
    // the global loads of the next group are issued into registers before the
    // interface arithmetic of the current one, so their latency overlaps it; with more
    // points per thread the extra registers would halve the occupancy, so the loads
    // stay at the top of each group.
    constexpr bool kPrefetch = P == 1;
    T pw[P][5], pg[P][4];
    auto fetch = [&](long long vb) {
        const int bi = find_box(L.off, L.nbox, vb);
        const BoxDesc &bx = L.boxes[bi];
        const int nx = bx.nx;
        const long long nrows = (long long)bx.ny * bx.nz;
        const long long row0 = (vb - L.off[bi]) * bx.rows;
        const int nact = (int)min((long long)bx.rows, nrows - row0) * nx;
        const size_t obase = (size_t)row0 * nx, n3 = bx.n3;
        const gptr<const T> u = glob((const T *)state_ptr(bx, L, L.in));
        const gptr<const T> G = glob((const T *)bx.G);
#pragma unroll
        for (int k = 0; k < P; ++k) {
            const int t = threadIdx.x + k * kRowThreads;
            if (t < nact) {
                const size_t o = obase + t;
#pragma unroll
                for (int v = 0; v < 5; ++v) pw[k][v] = u[v * n3 + o];
                if constexpr (VISC) {
                    pg[k][0] = load_g<0, 0>(G, n3, o);
                    pg[k][1] = load_g<0, 1>(G, n3, o);
                    pg[k][2] = load_g<0, 2>(G, n3, o);
                    pg[k][3] = load_g<0, 3>(G, n3, o);
                }
            }
        }
    };
    const VbRange R = vb_range(L.total);
    if (kPrefetch && R.vb < R.end) fetch(R.vb);
    for (long long vb = R.vb; vb < R.end; vb += R.stride) {
        const int bi = find_box(L.off, L.nbox, vb);
        const BoxDesc &bx = L.boxes[bi];
        const int nx = bx.nx;
        // LDS stride of a field: the block's points, or with one point per thread (every
        // block of rows fits 256 points) the constant 256, which turns the component
        // offsets of the stencil reads into immediates
        const int per = P == 1 ? kRowThreads : bx.rows * nx;
        T *su = lds;           // [5][per] states, later the interface fluxes
        T *sf = su + 5 * per;  // [5][per] point fluxes
        T *sg = sf + 5 * per;  // [4][per] viscous fluxes (VISC)
        const size_t n3 = bx.n3;
        const T gamma = T(bx.gamma), eps4 = T(4.0 * bx.eps), delta = T(bx.delta);
        const T gm1 = gamma - T(1);
        const T inv_dx = T(bx.inv_h[0]);
        const long long nrows = (long long)bx.ny * bx.nz;
        const long long row0 = (vb - L.off[bi]) * bx.rows;
        const int nact = (int)min((long long)bx.rows, nrows - row0) * nx;  // active points
        const size_t obase = (size_t)row0 * nx;
        const gptr<T> out = glob((T *)(L.out_ov ? L.out_ov : bx.rhs));

#pragma unroll
        for (int k = 0; k < P; ++k) {
            const int t = threadIdx.x + k * kRowThreads;
            if (t < nact) {
                T wk[5], gk[4], f[5];
                if constexpr (kPrefetch) {
#pragma unroll
                    for (int v = 0; v < 5; ++v) wk[v] = pw[k][v];
#pragma unroll
                    for (int c = 0; c < 4; ++c) gk[c] = pg[k][c];
                } else {
                    const gptr<const T> u = glob((const T *)state_ptr(bx, L, L.in));
                    const gptr<const T> G = glob((const T *)bx.G);
                    const size_t o = obase + t;
#pragma unroll
                    for (int v = 0; v < 5; ++v) wk[v] = u[v * n3 + o];
                    if constexpr (VISC) {
                        gk[0] = load_g<0, 0>(G, n3, o);
                        gk[1] = load_g<0, 1>(G, n3, o);
                        gk[2] = load_g<0, 2>(G, n3, o);
                        gk[3] = load_g<0, 3>(G, n3, o);
                    }
                }
                euler_flux5<T, 0>(wk, gm1, f);
#pragma unroll
                for (int v = 0; v < 5; ++v) {
                    su[v * per + t] = wk[v];
                    sf[v * per + t] = f[v];
                }
                if constexpr (VISC) {
#pragma unroll
                    for (int c = 0; c < 4; ++c) sg[c * per + t] = gk[c];
                }
            }
        }
        __syncthreads();
        if (kPrefetch && vb + R.stride < R.end) fetch(vb + R.stride);
        T H[P][5];
#pragma unroll
        for (int k = 0; k < P; ++k) {
            const int t = threadIdx.x + k * kRowThreads;
            if (t < nact) {
                const int r = t / nx, i = t - r * nx, rb = r * nx;
                int q[6];
#pragma unroll
                for (int m = 0; m < 6; ++m) q[m] = rb + wrapi(i - 2 + m, nx);
                interface_flux_lds<T, B, 0, VISC, WW>(su, sf, sg, per, q, gamma, eps4, delta, H[k]);  // at i+1/2
            }
        }
        __syncthreads();  // every thread has read the staged states
#pragma unroll
        for (int k = 0; k < P; ++k) {
            const int t = threadIdx.x + k * kRowThreads;
            if (t < nact)
#pragma unroll
                for (int v = 0; v < 5; ++v) su[v * per + t] = H[k][v];
        }
        __syncthreads();
#pragma unroll
        for (int k = 0; k < P; ++k) {
            const int t = threadIdx.x + k * kRowThreads;
            if (t < nact) {
                const int r = t / nx, i = t - r * nx;
                const int qm = r * nx + wrapi(i - 1, nx);
                const size_t o = obase + t;
#pragma unroll
                for (int v = 0; v < 5; ++v) out[v * n3 + o] = -(H[k][v] - su[v * per + qm]) * inv_dx;
            }
        }
        __syncthreads();  // LDS is reused by the next virtual block
    }
}

// ----------------------------------------------------------------------------
// x sweep for rows longer than a block: one block walks one periodic row in chunks of
// kRowThreads interfaces.  Chunk c stages the points c*256-2 .. c*256+258 (the six-point
// stencils of its interfaces, wrapped) in LDS and one thread forms one interface flux.
// The flux difference of point i takes the interface fluxes at i-1/2 and i+1/2; the first
// point of a chunk takes i-1/2 from the previous chunk (carried in LDS), and the row's
// first point waits for the last chunk.  Compared with staging the whole row, the LDS of
// a block does not grow with the row (15 KB), so the CU holds twice the blocks
// at 512 points per row; each chunk re-reads five stencil points of its neighbour.
// ----------------------------------------------------------------------------
constexpr int kChunkPts = kRowThreads + 5;  // points staged per chunk
__host__ __device__ __forceinline__ size_t chunk_lds_bytes(size_t esz) { return (14 * kChunkPts + 5) * esz; }

template <typename T, typename B, bool VISC, int WW>
__global__ __launch_bounds__(kRowThreads)
__attribute__((amdgpu_waves_per_eu(2))) void k_sweep_x_chunks(Launch L0) {
    const Launch L = with_params(L0);
    extern __shared__ unsigned char lds_raw[];
    T *su = reinterpret_cast<T *>(lds_raw);  // [5][kChunkPts] states, later the interface fluxes
    T *sf = su + 5 * kChunkPts;              // [5][kChunkPts] point fluxes
    T *sg = sf + 5 * kChunkPts;              // [4][kChunkPts] viscous fluxes (VISC)
    T *carry = sg + 4 * kChunkPts;           // [5] interface flux carried to the next chunk
    const int t = threadIdx.x;
    const VbRange R = vb_range(L.total);
    for (long long vb = R.vb; vb < R.end; vb += R.stride) {
        const int bi = find_box(L.off, L.nbox, vb);
        const BoxDesc &bx = L.boxes[bi];
        const int nx = bx.nx;
        const size_t n3 = uni64(bx.n3), obase = (size_t)(vb - L.off[bi]) * nx;
        const gptr<const T> u = uni(glob((const T *)state_ptr(bx, L, L.in)));
        const gptr<const T> G = uni(glob((const T *)bx.G));
        const gptr<T> out = uni(glob((T *)(L.out_ov ? L.out_ov : bx.rhs)));
        const T gamma = T(bx.gamma), eps4 = T(4.0 * bx.eps), delta = T(bx.delta);
        const T gm1 = gamma - T(1);
        const T inv_dx = T(bx.inv_h[0]);
        const int nch = (nx + kRowThreads - 1) / kRowThreads;
        T Hfirst[5];  // interface 1/2 of the row (thread 0)
        for (int c = 0; c < nch; ++c) {
            const int i0 = c * kRowThreads;
            for (int sp = t; sp < kChunkPts; sp += kRowThreads) {
                const size_t o = obase + wrapm(i0 - 2 + sp, nx);
                T wk[5], f[5];
#pragma unroll
                for (int v = 0; v < 5; ++v) wk[v] = u[v * n3 + o];
                euler_flux5<T, 0>(wk, gm1, f);
#pragma unroll
                for (int v = 0; v < 5; ++v) {
                    su[v * kChunkPts + sp] = wk[v];
                    sf[v * kChunkPts + sp] = f[v];
                }
                if constexpr (VISC) {
                    sg[0 * kChunkPts + sp] = load_g<0, 0>(G, n3, o);
                    sg[1 * kChunkPts + sp] = load_g<0, 1>(G, n3, o);
                    sg[2 * kChunkPts + sp] = load_g<0, 2>(G, n3, o);
                    sg[3 * kChunkPts + sp] = load_g<0, 3>(G, n3, o);
                }
            }
            __syncthreads();
            const int i = i0 + t;
            const bool act = i < nx;
            T H[5];
            if (act) {
                int q[6];
#pragma unroll
                for (int m = 0; m < 6; ++m) q[m] = t + m;  // point i-2+m
                interface_flux_lds<T, B, 0, VISC, WW>(su, sf, sg, kChunkPts, q, gamma, eps4, delta, H);  // at i+1/2
            }
            __syncthreads();  // every thread has read the staged chunk
            if (act)
#pragma unroll
                for (int v = 0; v < 5; ++v) su[v * kChunkPts + t] = H[v];
            if (c == 0 && t == 0)
#pragma unroll
                for (int v = 0; v < 5; ++v) Hfirst[v] = H[v];
            __syncthreads();
            // point i from the interfaces at i-1/2 and i+1/2; the row's first point waits
            if (act && (c > 0 || t > 0)) {
                const size_t o = obase + i;
#pragma unroll
                for (int v = 0; v < 5; ++v) {
                    const T hm = t > 0 ? su[v * kChunkPts + t - 1] : carry[v];
                    out[v * n3 + o] = -(H[v] - hm) * inv_dx;
                }
            }
            __syncthreads();  // carry read; the next chunk overwrites the staging
            if (i == min(i0 + kRowThreads, nx) - 1)
#pragma unroll
                for (int v = 0; v < 5; ++v) carry[v] = H[v];
        }
        __syncthreads();  // carry now holds the interface at nx-1/2
        if (t == 0) {
#pragma unroll
            for (int v = 0; v < 5; ++v) out[v * n3 + obase] = -(Hfirst[v] - carry[v]) * inv_dx;
        }
        __syncthreads();  // LDS is reused by the next row
    }
}

// ----------------------------------------------------------------------------
// launchers
// ----------------------------------------------------------------------------
int rows_for(int nx) {
    int g = 1;
    while (nx * g * 2 <= kRowThreads) g *= 2;
    return g;
}

int rows_points(int nx, int rows) { return (int)cdiv((long long)rows * nx, kRowThreads); }

void visc_fields(const Batch &bt, Launch L) {
    L = with_family(bt, L, F_VISC);
    if (!L.total) return;
    ProfScope ps(bt.prof, K_VISC_FLUX, bt.stream);
    hipLaunchKernelGGL((k_visc_flux<float>), dim3(grid_of(bt, F_VISC, L.total)), dim3(kPointThreads), 0, bt.stream, L);
}

void viscous(const Batch &bt, Launch L) {
    visc_fields(bt, L);
    L = with_family(bt, L, F_POINT);
    hipLaunchKernelGGL(k_visc_div<float>, dim3(grid_for(L.total)), dim3(kPointThreads), 0, bt.stream, L);
}

template <int DIR, int MODE, bool VISC>
static void sweep_t(const Batch &bt, const Launch &L) {
    const dim3 g(grid_of(bt, F_SWEEP_X + DIR, L.total)), b(bt.block);
    const size_t ring = 30 * (size_t)bt.block * sizeof(float);  // point-flux ring, 6 slots x 5 per thread
    if (bt.weights == CNS_WENO_Z)
        hipLaunchKernelGGL((k_sweep<float, double, DIR, MODE, VISC, CNS_WENO_Z>), g, b, ring, bt.stream, L);
    else if (bt.weights == CNS_WENO_M)
        hipLaunchKernelGGL((k_sweep<float, double, DIR, MODE, VISC, CNS_WENO_M>), g, b, ring, bt.stream, L);
    else
        hipLaunchKernelGGL((k_sweep<float, double, DIR, MODE, VISC, CNS_WENO_JS>), g, b, ring, bt.stream, L);
}

template <int MODE>
static void sweep(const Batch &bt, Launch L, int dir, bool visc) {
    L = with_family(bt, L, F_SWEEP_X + dir);
    if (!L.total) return;
    if (visc) {
        if (dir == 0) sweep_t<0, MODE, true>(bt, L);
        else if (dir == 1) sweep_t<1, MODE, true>(bt, L);
        else sweep_t<2, MODE, true>(bt, L);
    } else {
        if (dir == 0) sweep_t<0, MODE, false>(bt, L);
        else if (dir == 1) sweep_t<1, MODE, false>(bt, L);
        else sweep_t<2, MODE, false>(bt, L);
    }
}
void sweep_write(const Batch &bt, const Launch &L, int dir, bool visc) { sweep<MODE_WRITE>(bt, L, dir, visc); }
void sweep_accum(const Batch &bt, const Launch &L, int dir, bool visc) { sweep<MODE_ACCUM>(bt, L, dir, visc); }
void sweep_rk(const Batch &bt, const Launch &L, bool visc) { sweep<MODE_RK>(bt, L, 2, visc); }

template <bool VISC, int WW>
static void xrows_tw(const Batch &bt, const Launch &L) {
    // about four row groups per block when the loads of the next one are prefetched
    const long long nb = bt.grid[F_XROWS] > 0 ? std::min<long long>(bt.grid[F_XROWS], L.total)
                         : (bt.rowP == 1 ? std::max<long long>(std::min<long long>(L.total, 2048), L.total / 4)
                                         : L.total);
    const dim3 g(grid_for(nb)), b(kRowThreads);
    switch (bt.rowP) {
        case 1: hipLaunchKernelGGL((k_sweep_x_rows<float, double, VISC, 1, WW>), g, b, bt.rowLds, bt.stream, L); break;
        case 2: hipLaunchKernelGGL((k_sweep_x_rows<float, double, VISC, 2, WW>), g, b, bt.rowLds, bt.stream, L); break;
        case 3: hipLaunchKernelGGL((k_sweep_x_rows<float, double, VISC, 3, WW>), g, b, bt.rowLds, bt.stream, L); break;
        default: hipLaunchKernelGGL((k_sweep_x_rows<float, double, VISC, 4, WW>), g, b, bt.rowLds, bt.stream, L); break;
    }
}

template <bool VISC>
static void xrows_t(const Batch &bt, const Launch &L) {
    if (bt.weights == CNS_WENO_Z) xrows_tw<VISC, CNS_WENO_Z>(bt, L);
    else if (bt.weights == CNS_WENO_M) xrows_tw<VISC, CNS_WENO_M>(bt, L);
    else xrows_tw<VISC, CNS_WENO_JS>(bt, L);
}

template <bool VISC>
static void xchunks_t(const Batch &bt, const Launch &L) {
    const dim3 g(grid_of(bt, F_XCHUNK, L.total)), b(kRowThreads);
    const size_t lds = chunk_lds_bytes(sizeof(float));
    if (bt.weights == CNS_WENO_Z)
        hipLaunchKernelGGL((k_sweep_x_chunks<float, double, VISC, CNS_WENO_Z>), g, b, lds, bt.stream, L);
    else if (bt.weights == CNS_WENO_M)
        hipLaunchKernelGGL((k_sweep_x_chunks<float, double, VISC, CNS_WENO_M>), g, b, lds, bt.stream, L);
    else
        hipLaunchKernelGGL((k_sweep_x_chunks<float, double, VISC, CNS_WENO_JS>), g, b, lds, bt.stream, L);
}

void sweep_x(const Batch &bt, const Launch &L, bool visc) {
    ProfScope ps(bt.prof, K_SWEEP_X, bt.stream);
    const Launch R = with_family(bt, L, F_XROWS);
    if (R.total) {
        if (visc) xrows_t<true>(bt, R);
        else xrows_t<false>(bt, R);
    }
    const Launch C = with_family(bt, L, F_XCHUNK);
    if (C.total) {
        if (visc) xchunks_t<true>(bt, C);
        else xchunks_t<false>(bt, C);
    }
    sweep<MODE_WRITE>(bt, L, 0, visc);
}

int resident_sweep_blocks(int block) {
    int n = 0;
    const hipError_t e = hipOccupancyMaxActiveBlocksPerMultiprocessor(
        &n, k_sweep<float, double, 2, MODE_RK, true, CNS_WENO_JS>, block, 30 * (size_t)block * sizeof(float));
    return e == hipSuccess ? n : 0;
}
int resident_tile_blocks() {
    int n = 0;
    const hipError_t e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, k_visc_flux<float>, kPointThreads, 0);
    return e == hipSuccess ? n : 0;
}

}  // namespace mixed
}  // namespace cns
