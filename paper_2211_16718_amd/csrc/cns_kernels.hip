// cns_kernels.hip -- gfx950 kernels of the WENO5-Roe / central-viscous RHS and RK4.
//
// Data layout in HBM: SoA state u[v][k][j][i] (x fastest) per box.  One RHS
// evaluation of a batch of boxes is
//   1. k_visc       : u -> the viscous and heat-flux terms sum_d D_d G_d of the momentum
//                     and energy equations [4][N3] (skipped when mu_eff = 0)
//   2. x sweep      : u, viscous terms -> rhs (write).  Rows staged in LDS, two cells per
//                     thread (k_sweep_x_rows; k_sweep_x_chunks for rows above 512 points)
//   3. k_sweep<y>   : u -> rhs (accumulate)
//   4. k_sweep<z>   : u -> rhs (accumulate), or the fused Runge-Kutta stage update.
// A marching thread owns a segment of one grid line and walks along it cell by cell:
// every point flux, every cell's face values and every interface flux is formed once
// per segment, the flux difference in registers.  FP64; the mixed form has its own
// kernels for 1 to 4 (cns_mixed.hip).
// Periodic boundaries wrap the line index; there are no ghost cells.
//
// Every kernel takes a Launch over a batch of boxes (see cns_internal.h) and loops
// over virtual blocks, so one launch advances every box of an ensemble.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <type_traits>

#include "cns_batch.h"
#include "cns_mixed.h"

namespace cns {

// ----------------------------------------------------------------------------
// state from primitives (Sec. 2.1 equation of state); single box
// ----------------------------------------------------------------------------
template <typename T>
__global__ void k_init_state(size_t n3, double gm1, const double *rho, const double *vel, const double *p, T *u) {
    size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x;
    if (i >= n3) return;
    double r = rho[i], a = vel[i], b = vel[n3 + i], c = vel[2 * n3 + i];
    u[i] = T(r);
    u[n3 + i] = T(r * a);
    u[2 * n3 + i] = T(r * b);
    u[3 * n3 + i] = T(r * c);
    u[4 * n3 + i] = T(p[i] / gm1 + 0.5 * r * (a * a + b * b + c * c));
}

template <typename T>
__global__ void k_fill(size_t n, T *out) {
    size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x;
    if (i < n) out[i] = T(0);
}

// ----------------------------------------------------------------------------
// viscous terms: primitives, then viscous fluxes at points
// ----------------------------------------------------------------------------
// The 5-point central difference (times 12 h): the viscous kernel states every fused
// multiply-add itself (contraction off), so that its variant that also accumulates the
// diagnostics (extra uses of the gradients) gives the same bits.
__device__ __forceinline__ double vfma(double a, double b, double c) { return fma(a, b, c); }
__device__ __forceinline__ float vfma(float a, float b, float c) { return fmaf(a, b, c); }
template <typename T>
__device__ __forceinline__ T dcen12(T m2, T m1, T p1, T p2) {
#pragma clang fp contract(off)
    return vfma(T(8), p1 - m1, m2 - p2);
}

// primitives (u, v, w, T = gamma p / rho) of a loaded state
template <typename T>
__device__ __forceinline__ void prim_of(const T s[5], T gamma, T W[4]) {
#pragma clang fp contract(off)
    const T inv = rcp(s[0]);
    W[0] = s[1] * inv;
    W[1] = s[2] * inv;
    W[2] = s[3] * inv;
    const T p = (gamma - T(1)) * (s[4] - T(0.5) * (s[1] * W[0] + s[2] * W[1] + s[3] * W[2]));
    W[3] = gamma * p * inv;
}

// The point quantities of the diagnostics of a loaded state with primitives W: kinetic
// energy, mass, momentum, energy, the largest wave speed and the bad-point count in acc;
// returns whether the point is valid (finite, rho > 0, p > 0).
__device__ __forceinline__ bool prim_stats(const double s[5], const double W[4], double gamma, double acc[CNS_NDIAG]) {
#pragma clang fp contract(off)
    const double r = s[0], mx = s[1], my = s[2], mz = s[3], e = s[4];
    const double inv = rcp(r);
    const double ke = 0.5 * fma(mz, W[2], fma(my, W[1], mx * W[0]));
    const double p = (gamma - 1.0) * (e - ke);
    const bool finite = isfinite(r) && isfinite(mx) && isfinite(my) && isfinite(mz) && isfinite(e);
    if (!finite || !(r > 0.0) || !(p > 0.0)) {
        acc[8] += 1.0;
        return false;
    }
    acc[0] += ke;
    acc[2] += r;
    acc[3] += mx;
    acc[4] += my;
    acc[5] += mz;
    acc[6] += e;
    const double c = sqrt(gamma * p * inv);
    acc[7] = fmax(acc[7], fmax(fabs(W[0]), fmax(fabs(W[1]), fabs(W[2]))) + c);
    return true;
}
template <int NW>
__device__ __forceinline__ void block_reduce_diag(const double acc[CNS_NDIAG], double (*red)[CNS_NDIAG],
                                                  gptr<double> dst, unsigned mask);

// The staging box of a viscous tile has its origin at (x0 - 4, y0 - 4).  Its halo points,
// where the tile's outer derivatives need viscous fluxes: rows y0-2, y0-1, y0+TY, y0+TY+1
// of the tile's columns (kHaloY of them, whole waves), then columns x0-2, x0-1, x0+TX,
// x0+TX+1 of its rows: the y and the x halo need different fluxes, and no wave has both.
// Further points, whose primitives the gradients of the halo points need: the 2 x 2
// corners between the halos, then columns x0-4, x0-3, x0+TX+2, x0+TX+3 of the tile's rows,
// then rows y0-4, y0-3, y0+TY+2, y0+TY+3 of its columns.
template <typename T>
struct ViscTile {
    static constexpr int TX = kViscTX, TY = kViscTY, kThreads = TX * TY;
    static constexpr int kHaloY = 4 * TX, kHalo = kHaloY + 4 * TY, kExt = 16 + 4 * TY + 4 * TX;
    static_assert(kHaloY % 64 == 0, "no wave holds points of both halos");
    static_assert(kHalo <= kThreads && kExt <= kThreads, "one halo and one further point per thread");
    static __device__ __forceinline__ void halo_pos(int h, int &bx, int &by) {
        if (h < kHaloY) {
            const int r = h / TX;
            bx = 4 + h % TX;
            by = r < 2 ? 2 + r : TY + 2 + r;
        } else {
            const int q = h - kHaloY, c = q & 3;
            bx = c < 2 ? 2 + c : TX + 2 + c;
            by = 4 + (q >> 2);
        }
    }
    static __device__ __forceinline__ void ext_pos(int e, int &bx, int &by) {
        if (e < 16) {
            const int cc = e >> 2;
            bx = (cc & 1 ? TX + 4 : 2) + (e & 1);
            by = (cc & 2 ? TY + 4 : 2) + ((e >> 1) & 1);
        } else if (e < 16 + 4 * TY) {
            const int q = e - 16, c = q & 3;
            bx = c < 2 ? c : TX + 4 + c;
            by = 4 + (q >> 2);
        } else {
            const int q = e - 16 - 4 * TY, r = q / TX;
            bx = 4 + q % TX;
            by = r < 2 ? r : TY + 4 + r;
        }
    }
};

// Viscous and heat-flux terms: vd = sum_d D_d G_d, the viscous fluxes G formed and
// differentiated in one pass (primitives -> 12 first derivatives -> tau, q -> G -> vd).
// A block owns a 32 x 8 (x, y) tile and marches along z over vsz planes.  Each
// thread keeps its own column's primitives at planes k-2 .. k+2 in registers; per plane
// the block stages the primitives of the tile and of its +-4 halo in LDS, every thread
// forms the gradients and G of its point, the owners of the halo points also those of
// their halo point (z derivatives from their own LDS ring of five planes), G_x and G_y
// meet in LDS, and G_z enters the pending sums of the planes k-2 .. k+2.  G is formed
// at 1.6 points per point of the tile and at 4 extra planes per block, but never goes
// through memory: 9 fields written and 12 read by the sweeps become 4 written and 4 read.
// Every plane's sum takes its terms in the same order wherever a block starts.  Each load
// is issued one plane ahead of its use, and five planes per pass rotate the windows by
// renaming registers.
// 512^3: 3.95 ms against 3.29 ms for the nine fluxes alone, whose 12 reads then cost each
// sweep 0.9 ms more.  LDS half busy, VALU 0.4, 4.5 TB/s with the halos: the two barriers
// per plane leave none saturated.  Tiles of 16 x 16 with a thread per halo column took 6.4 ms
// (bank conflicts), of 32 x 16 the same time at 512^3 and 8 % more on ragged boxes.
//
// With DIAG (FP64 plans, the first stage of a step) the kernel also forms the partial
// diagnostics of the state it reads, one partial per tile and group of diag_planes planes:
// the point quantities of a plane as its column is loaded, the enstrophy from the velocity
// gradients it computes anyway (the same central derivatives as the diagnostics kernel).  The state's
// diagnostics then cost no read of their own.
template <typename T, bool DIAG>
struct ViscLds {
    using Tile = ViscTile<T>;
    static constexpr int TX = Tile::TX, TY = Tile::TY;
    T sW[4][TY + 8][TX + 8];  // primitives of the plane, origin (x0-4, y0-4)
    T sFx[4][TY][TX + 4];     // G_x on the tile's rows and their x halo
    T sFy[4][TY + 4][TX];     // G_y on the tile's columns and their y halo
    T hW[5][4][Tile::kHalo];  // primitives of the halo points, planes k-2 .. k+2
    double red[DIAG ? Tile::kThreads / 64 : 1][CNS_NDIAG];
};
template <typename T, bool DIAG>
__device__ __forceinline__ void visc_blocks(const Launch &L, const VbRange R, ViscLds<T, DIAG> &S) {
#pragma clang fp contract(off)
    static_assert(!DIAG || std::is_same<T, double>::value, "fused diagnostics in FP64 plans only");
    using Tile = ViscTile<T>;
    constexpr int TX = Tile::TX, TY = Tile::TY, kVThreads = Tile::kThreads, kVh = Tile::kHalo;
    auto &sW = S.sW;
    auto &sFx = S.sFx;
    auto &sFy = S.sFy;
    auto &hW = S.hW;
    auto &red = S.red;
    const int tx = threadIdx.x % TX, ty = threadIdx.x / TX;
    for (long long vb = R.vb; vb < R.end; vb += R.stride) {
        const int bi = find_box(L.off, L.nbox, vb);
        const BoxDesc &b = L.boxes[bi];
        const int nx = b.nx, ny = b.ny, nz = b.nz;
        const size_t n3 = uni64(b.n3), sz = (size_t)nx * ny;
        const long long lb = vb - L.off[bi];
        // the halo points fall to the first waves of a block or, in every other set of 32 blocks
        // (one per CU of an XCD), to the last: the two blocks of a CU load its SIMDs evenly
        const int h = (threadIdx.x + (lb & 32 ? kVThreads / 2 : 0)) % kVThreads, e = kVThreads - 1 - h;
        const bool own_h = h < kVh, yhalo = h < Tile::kHaloY, own_e = e < Tile::kExt;
        int hbx = 0, hby = 0, ebx = 0, eby = 0;
        if (own_h) Tile::halo_pos(h, hbx, hby);
        if (own_e) Tile::ext_pos(e, ebx, eby);
        const int ntx = (nx + TX - 1) / TX, nty = (ny + TY - 1) / TY;
        const int x0 = (int)(lb % ntx) * TX, y0 = (int)((lb / ntx) % nty) * TY;
        const int vsz = L.vsz_ov ? L.vsz_ov : b.vsz;
        const int z0 = (int)(lb / ((long long)ntx * nty)) * vsz, z1 = min(z0 + vsz, nz);
        const bool act = x0 + tx < nx && y0 + ty < ny;
        // a column past a ragged edge wraps periodically: its primitives are halo values
        // of the active columns beside it
        const uint32_t col = (uint32_t)(wrapm(y0 + ty, ny) * nx + wrapm(x0 + tx, nx));
        const uint32_t hcol = (uint32_t)(wrapm(y0 - 4 + hby, ny) * nx + wrapm(x0 - 4 + hbx, nx));
        const uint32_t ecol = (uint32_t)(wrapm(y0 - 4 + eby, ny) * nx + wrapm(x0 - 4 + ebx, nx));
        const gptr<const T> u = uni(glob((const T *)state_ptr(b, L, L.in)));
        const gptr<T> out = uni(glob(L.v_ov ? (T *)L.v_ov : (T *)b.G));
        const T gamma = T(b.gamma);
        // the 1/12 of the central differences is folded into the spacings
        const T ihx = T(b.inv_h[0] / 12.0), ihy = T(b.inv_h[1] / 12.0), ihz = T(b.inv_h[2] / 12.0);
        const T mu = T(b.mu), kcond = T(b.mu / ((b.gamma - 1.0) * b.prandtl));
        auto load = [&](uint32_t c, int plane, T s[5]) {
            const uint32_t bo = (uint32_t)((c + (size_t)wrapi(plane, nz) * sz) * sizeof(T));
#pragma unroll
            for (int v = 0; v < 5; ++v) s[v] = *elem(u, n3, v, bo);
        };
        // windows over the planes k-2 .. k+2, plane k-2+m in slot (r+m) mod 5 at step r of a pass
        T Wz[5][4];  // this column's primitives
        T Tq[5][4];  // vd of this column as it accumulates
        double acc[CNS_NDIAG] = {0, 0, 0, 0, 0, 0, 0, 0, 0};
        unsigned good = 0;  // bit m: the column's point at plane k-2+m is valid (DIAG)
        const int k0 = z0 - 2;
        // the sums of a group leave for the partials of its tile: the point quantities once its
        // last plane has entered, the enstrophy once its last plane is formed
        const int grp = diag_planes(nx, ny, nz);
        auto flush = [&](int plane, bool enstrophy) {
            if constexpr (DIAG) {
                const gptr<double> dst = glob(b.part) + (lb % ((long long)ntx * nty) +
                                                         (long long)ntx * nty * (plane / grp)) * CNS_NDIAG;
                block_reduce_diag<kVThreads / 64>(acc, red, dst, enstrophy ? 2u : ~2u);
#pragma unroll
                for (int d = 0; d < CNS_NDIAG; ++d)
                    if ((d == 1) == enstrophy) acc[d] = 0.0;
            }
        };
        auto enter = [&](const T s[5], int plane, int slot, int m) {
            prim_of(s, gamma, Wz[slot]);
            if constexpr (DIAG) {
                if (plane > z0 && plane <= z1 && (plane == z1 || plane % grp == 0)) flush(plane - 1, false);
                if (act && plane >= z0 && plane < z1 && prim_stats(s, Wz[slot], gamma, acc)) good |= 1u << m;
            }
        };
#pragma unroll
        for (int m = 0; m < 5; ++m) {
            T s[5];
            load(col, k0 - 2 + m, s);
            enter(s, k0 - 2 + m, m, m);
#pragma unroll
            for (int c = 0; c < 4; ++c) Tq[m][c] = T(0);
        }
        if (own_h)
#pragma unroll
            for (int m = 0; m < 5; ++m) {
                T s[5], w4[4];
                load(hcol, k0 - 2 + m, s);
                prim_of(s, gamma, w4);
#pragma unroll
                for (int c = 0; c < 4; ++c) hW[m][c][h] = w4[c];
            }
        T es[5] = {T(1), T(0), T(0), T(0), T(0)};  // state of the further point at the next full plane
        auto step = [&](auto rc, const int k) {
#pragma clang fp contract(off)
            constexpr int r = decltype(rc)::value;
            constexpr int i0 = r % 5, i1 = (r + 1) % 5, i2 = (r + 2) % 5, i3 = (r + 3) % 5, i4 = (r + 4) % 5;
            // planes z0 .. z1-1 are formed in full; the two planes on either side only for G_z
            const bool full = k >= z0 && k < z1;
            T cs[5], hs[5];  // plane k+3 of the column and of the halo point
            load(col, k + 3, cs);
            if (own_h) {
                load(hcol, k + 3, hs);
#pragma unroll
                for (int c = 0; c < 4; ++c) sW[c][hby][hbx] = hW[i2][c][h];
            }
            if (own_e) {
                if (full) {
                    T w4[4];
                    prim_of(es, gamma, w4);
#pragma unroll
                    for (int c = 0; c < 4; ++c) sW[c][eby][ebx] = w4[c];
                }
                if (k + 1 >= z0 && k + 1 < z1) load(ecol, k + 1, es);
            }
#pragma unroll
            for (int c = 0; c < 4; ++c) sW[c][ty + 4][tx + 4] = Wz[i2][c];
            __syncthreads();
            // derivatives of field a at box position (X, Y)
            auto ddx = [&](int a, int X, int Y) {
                return dcen12(sW[a][Y][X - 2], sW[a][Y][X - 1], sW[a][Y][X + 1], sW[a][Y][X + 2]) * ihx;
            };
            auto ddy = [&](int a, int X, int Y) {
                return dcen12(sW[a][Y - 2][X], sW[a][Y - 1][X], sW[a][Y + 1][X], sW[a][Y + 2][X]) * ihy;
            };
            {
                T g[4][3];  // gradients of (u, v, w, T)
#pragma unroll
                for (int a = 0; a < 4; ++a) {
                    g[a][0] = ddx(a, tx + 4, ty + 4);
                    g[a][1] = ddy(a, tx + 4, ty + 4);
                    g[a][2] = dcen12(Wz[i0][a], Wz[i1][a], Wz[i3][a], Wz[i4][a]) * ihz;
                }
                if constexpr (DIAG) {
                    if (full && (good & 4u)) {
                        // vorticity of the velocity, as the diagnostics kernel forms it
                        const double ox = g[2][1] - g[1][2], oy = g[0][2] - g[2][0], oz = g[1][0] - g[0][1];
                        if (isfinite(ox) && isfinite(oy) && isfinite(oz)) acc[1] = fma(0.5, fma(oz, oz, fma(oy, oy, ox * ox)), acc[1]);
                    }
                    if (full && (k + 1 == z1 || (k + 1) % grp == 0)) flush(k, true);
                }
                const T vx = Wz[i2][0], vy = Wz[i2][1], vz = Wz[i2][2];
                const T tdiv = (T(2) / T(3)) * ((g[0][0] + g[1][1]) + g[2][2]);
                const T txz = mu * (g[0][2] + g[2][0]), tyz = mu * (g[1][2] + g[2][1]);
                const T tzz = mu * vfma(T(2), g[2][2], -tdiv);
                const T Gz[4] = {txz, tyz, tzz, vfma(vx, txz, vfma(vy, tyz, vfma(vz, tzz, kcond * g[3][2])))};
                // D_z G_z: dcen = (8 (p1 - m1) - (p2 - m2)) / 12, so G_z of this plane enters the
                // planes k-2, k-1, k+1, k+2 with -1, 8, -8, 1 times ihz
#pragma unroll
                for (int a = 0; a < 4; ++a) {
                    const T w = ihz * Gz[a];
                    Tq[i0][a] -= w;
                    Tq[i1][a] = vfma(T(8), w, Tq[i1][a]);
                    Tq[i3][a] = vfma(T(-8), w, Tq[i3][a]);
                    Tq[i4][a] = w;
                }
                if (full) {
                    const T txx = mu * vfma(T(2), g[0][0], -tdiv), tyy = mu * vfma(T(2), g[1][1], -tdiv);
                    const T txy = mu * (g[0][1] + g[1][0]);
                    sFx[0][ty][tx + 2] = txx;
                    sFx[1][ty][tx + 2] = txy;
                    sFx[2][ty][tx + 2] = txz;
                    sFx[3][ty][tx + 2] = vfma(vx, txx, vfma(vy, txy, vfma(vz, txz, kcond * g[3][0])));
                    sFy[0][ty + 2][tx] = txy;
                    sFy[1][ty + 2][tx] = tyy;
                    sFy[2][ty + 2][tx] = tyz;
                    sFy[3][ty + 2][tx] = vfma(vx, txy, vfma(vy, tyy, vfma(vz, tyz, kcond * g[3][1])));
                }
            }
            if (own_h && full) {
                // a halo point: the eight derivatives its G_y (y halo) or G_x (x halo) takes
                auto hdz = [&](int a) { return dcen12(hW[i0][a][h], hW[i1][a][h], hW[i3][a][h], hW[i4][a][h]) * ihz; };
                const T vx = sW[0][hby][hbx], vy = sW[1][hby][hbx], vz = sW[2][hby][hbx];
                const T ux = ddx(0, hbx, hby), vyy = ddy(1, hbx, hby), wz = hdz(2);
                const T tdiv = (T(2) / T(3)) * ((ux + vyy) + wz);
                const T txy = mu * (ddy(0, hbx, hby) + ddx(1, hbx, hby));
                if (yhalo) {
                    const T tyy = mu * vfma(T(2), vyy, -tdiv), tyz = mu * (hdz(1) + ddy(2, hbx, hby));
                    sFy[0][hby - 2][hbx - 4] = txy;
                    sFy[1][hby - 2][hbx - 4] = tyy;
                    sFy[2][hby - 2][hbx - 4] = tyz;
                    sFy[3][hby - 2][hbx - 4] =
                        vfma(vx, txy, vfma(vy, tyy, vfma(vz, tyz, kcond * ddy(3, hbx, hby))));
                } else {
                    const T txx = mu * vfma(T(2), ux, -tdiv), txz = mu * (hdz(0) + ddx(2, hbx, hby));
                    sFx[0][hby - 4][hbx - 2] = txx;
                    sFx[1][hby - 4][hbx - 2] = txy;
                    sFx[2][hby - 4][hbx - 2] = txz;
                    sFx[3][hby - 4][hbx - 2] =
                        vfma(vx, txx, vfma(vy, txy, vfma(vz, txz, kcond * ddx(3, hbx, hby))));
                }
            }
            __syncthreads();
            if (full) {
#pragma unroll
                for (int a = 0; a < 4; ++a) {
                    const T dx = dcen12(sFx[a][ty][tx], sFx[a][ty][tx + 1], sFx[a][ty][tx + 3], sFx[a][ty][tx + 4]);
                    const T dy = dcen12(sFy[a][ty][tx], sFy[a][ty + 1][tx], sFy[a][ty + 3][tx], sFy[a][ty + 4][tx]);
                    Tq[i2][a] = vfma(ihx, dx, vfma(ihy, dy, Tq[i2][a]));
                }
            }
            if (k - 2 >= z0 && act) {
                const uint32_t bo = (uint32_t)((col + (size_t)(k - 2) * sz) * sizeof(T));
#pragma unroll
                for (int a = 0; a < 4; ++a) __builtin_nontemporal_store(Tq[i0][a], elem(out, n3, a, bo));
            }
            // plane k+3 enters the windows in place of plane k-2
            good >>= 1;
            enter(cs, k + 3, i0, 4);
            if (own_h) {
                T w4[4];
                prim_of(hs, gamma, w4);
#pragma unroll
                for (int c = 0; c < 4; ++c) hW[i0][c][h] = w4[c];
            }
        };
        for (int k = k0;;) {
            step(std::integral_constant<int, 0>{}, k);
            if (++k >= z1 + 2) break;
            step(std::integral_constant<int, 1>{}, k);
            if (++k >= z1 + 2) break;
            step(std::integral_constant<int, 2>{}, k);
            if (++k >= z1 + 2) break;
            step(std::integral_constant<int, 3>{}, k);
            if (++k >= z1 + 2) break;
            step(std::integral_constant<int, 4>{}, k);
            if (++k >= z1 + 2) break;
        }
        // the next virtual block may give a halo point to another wave, which fills its ring
        // where this block's last step has just stored
        if (vb + R.stride < R.end) __syncthreads();
    }
}

template <typename T, bool DIAG>
__global__ __launch_bounds__(ViscTile<T>::kThreads, 2) void k_visc(Launch L0) {
    __shared__ ViscLds<T, DIAG> S;
    const Launch L = with_params(L0);
    visc_blocks<T, DIAG>(L, vb_range(L.total), S);
}

// ----------------------------------------------------------------------------
// marching WENO5-Roe sweep along one direction
// ----------------------------------------------------------------------------
// MODE_RAW: the flux differences themselves, for k_stage_sum.  MODE_RK1/2/3: the fused
// Runge-Kutta update, by what it reads besides rhs and the stage state: nothing (first stages),
// u^n, or u^n and the accumulator (RK4 stage 4).  One kernel with a run-time choice holds the
// operands of all three and spills 25 registers.
enum { MODE_WRITE = 0, MODE_ACCUM = 1, MODE_RK1 = 2, MODE_RK2 = 3, MODE_RK3 = 4, MODE_RAW = 5 };
constexpr bool is_rk(int mode) { return mode >= MODE_RK1 && mode <= MODE_RK3; }

// The update of one component at a point: kk the right-hand side, us the stage state, uo the
// state u^n and pa the accumulator (where MODE reads them); ue, ae their destinations.
// RK4: the FP64 stage states give back dt k1 / 6 = (U2 - u) / 3 and dt k3 / 3 = (U4 - u) / 3,
// so the accumulator is written in stage 2 and read in stage 4 only.  TVD-RK3 in Shu-Osher
// form: U1 = u + dt k; U2 = 3/4 u + 1/4 (U1 + dt k); u^{n+1} = 1/3 u + 2/3 (U2 + dt k).
template <int MODE, typename T>
__device__ __forceinline__ void rk_update(const Launch &L, double dt, double kk, double us, double uo, double pa,
                                          gptr<T> ue, gptr<double> ae) {
#pragma clang fp contract(off)
    if constexpr (MODE == MODE_RK1) {
        if (L.scheme == CNS_TVDRK3) *ue = T(fma(dt, kk, us));
        else *ue = T(fma(0.5 * dt, kk, us));
    } else if constexpr (MODE == MODE_RK2) {
        if (L.scheme == CNS_TVDRK3) {
            const double e = fma(dt, kk, us);
            if (L.stage == 2) *ue = T(fma(0.75, uo, 0.25 * e));
            else *ue = T(fma(1.0 / 3.0, uo, (2.0 / 3.0) * e));
        } else if (L.stage == 2) {
            __builtin_nontemporal_store(fma(dt / 3.0, kk, fma(1.0 / 3.0, us - uo, uo)), ae);
            *ue = T(fma(0.5 * dt, kk, uo));
        } else {
            *ue = T(fma(dt, kk, uo));
        }
    } else {
        *ue = fma(dt / 6.0, kk, fma(1.0 / 3.0, us - uo, pa));
    }
}

// Where the raw flux differences of a direction go: x to rhs, y to the planes of G that the
// viscous terms leave free, z to the stage buffer that is not this stage's input (also with
// the stage states elsewhere: the box's own buffers are then free).
template <typename T, int DIR>
__device__ __forceinline__ gptr<T> raw_buf(const BoxDesc &b, const Launch &L) {
    return glob((T *)(DIR == 0 ? b.rhs : (DIR == 1 ? (void *)((T *)b.G + 4 * b.n3) : (L.in == BUF_A ? b.B : b.A))));
}

// Lanes run over consecutive lines of the plane (coalesced).  For y, a block of W
// waves covers 64 lines times W consecutive segments, so neighbouring segments share
// their six-point halos in the CU's cache; for x and z a block covers 64 W lines of one
// segment (stacking z segments spreads a block over planes far apart in memory).
//
// A thread keeps the states of six consecutive points in registers and their fluxes 1-4
// in a ring in LDS (6 slots x 4 components, component-major across the wave so lanes hit
// distinct banks), read one component at a time; the sixth register slot receives the
// next point's load, issued a whole step ahead of its use, as are the loads of the output
// operands.  The step of cell k forms the cell's face values (weno5_cell6); those of its
// right face, and what the Roe average takes from the cell, are carried to the next step,
// those of its left face close the interface k-1/2, whose flux gives the difference at
// point k-1.  Three steps per pass, so the window rotates by renaming registers and by
// three slot copies a pass.
//
// Measured at 512^3 (interfaces formed from both biases, ten reconstructions and nine
// stored viscous fluxes before): y 5.38 -> 3.85 ms, 987 -> 700 VALU instructions per point
// and 20.9 -> 16.6 GB, now 0.81 of the issue slots at the 1.86 GHz the power limit leaves
// and 0.92 of the copy rate; z with the update 6.16 -> 4.85 ms (mean of the stages), 0.9-1.0
// of the copy rate: bound by memory.
template <typename T, int DIR, int MODE, bool VISC, int WW>
__device__ __forceinline__ void sweep_blocks(const Launch &L, const VbRange R, unsigned char *lds_raw) {
#pragma clang fp contract(off)
    // each wave's ring: slot s, component v of lane l at (s * 4 + v) * 64 + l, so the
    // component and slot strides are constants (immediate LDS offsets); slots 0-2 and 3-5
    // trade places after every pass
    constexpr int kSlot = 4 * 64;
    T *const ring0 = reinterpret_cast<T *>(lds_raw) + (threadIdx.x >> 6) * (6 * kSlot) + (threadIdx.x & 63);
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
        const int len = min(seg, n - j0);  // points of the segment
        const size_t n3 = uni64(bx.n3);
        const gptr<const T> u = uni(glob((const T *)state_ptr(bx, L, L.in)));
        const gptr<const T> vd = uni(glob((const T *)bx.G));
        const T eps4 = T(4.0 * bx.eps), delta = T(bx.delta);
        const T gm1 = T(bx.gamma) - T(1);
        const T inv_dx = T(bx.inv_h[DIR]);
        const double dt = L.dt_ov > 0.0 ? L.dt_ov : bx.dt;
        // Every pointer the loop uses is read from the box table here, once: the loop
        // stores to global memory, which the compiler cannot tell apart from the table, so
        // a table read inside the loop would be repeated after every store, each time
        // behind a wait for all loads in flight (the ones issued ahead included).
        const gptr<const T> rhs_in = uni(glob((const T *)(is_rk(MODE) ? bx.rhs : (L.out_ov ? L.out_ov : bx.rhs))));
        const gptr<const T> un = uni(glob((const T *)state_ptr(bx, L, BUF_U)));
        const gptr<double> acc = uni(glob(bx.acc));
        const gptr<T> unext = uni(glob((T *)state_ptr(bx, L, L.out)));
        const gptr<T> rhs_out = MODE == MODE_RAW ? uni(raw_buf<T, DIR>(bx, L))
                                                 : uni(glob((T *)(L.out_ov ? L.out_ov : bx.rhs)));

        T w[6][5];                // states: step r of a pass finds point k-2+m in w[r+m]
        T Lf[kNS];                // face values of cell k-1 at k-1/2
        RoeCell<T> ca;            // of cell k-1
        T Hp[5];                  // interface flux at k-3/2
        T *rlo = ring0, *rhi = ring0 + 3 * kSlot;
#pragma unroll
        for (int c = 0; c < kNS; ++c) Lf[c] = T(0);
        ca = RoeCell<T>{T(1), {T(0), T(0), T(0)}, T(1)};
        auto load = [&](int j, T (&d)[5]) {
            const uint32_t bo = (uint32_t)((base + wrapi(j, n) * sg.lstride) * sizeof(T));
#pragma unroll
            for (int v = 0; v < 5; ++v) d[v] = *elem(u, n3, v, bo);
        };
        // the step's ring slot of point k-2+m: r+m, modulo 6
        auto slot = [&](int s) -> T * { return s % 6 < 3 ? rlo + (s % 3) * kSlot : rhi + (s % 3) * kSlot; };
        auto put_flux = [&](int s, const T (&d)[5]) {
            T f[4];
            euler_flux<T, DIR>(d, gm1, f);
            T *o = slot(s);
#pragma unroll
            for (int v = 0; v < 4; ++v) o[v * 64] = f[v];
        };
#pragma unroll
        for (int m = 0; m < 5; ++m) load(j0 - 3 + m, w[m]);
#pragma unroll
        for (int m = 0; m < 4; ++m) put_flux(m, w[m]);
        // step i takes cell k = j0 - 1 + i, i = 0 .. len + 1
        auto step = [&](auto rc, const int i) {
#pragma clang fp contract(off)
            constexpr int r = decltype(rc)::value;
            const int k = j0 - 1 + i;
            // The window enters each step through an empty asm: otherwise the optimiser
            // shares the differences and indicator terms of a scalar between the cells of
            // a pass and holds them for all scalars at once (hundreds of spilled registers).
#pragma unroll
            for (int m = 0; m < 5; ++m)
#pragma unroll
                for (int v = 0; v < 5; ++v) pin(w[(r + m) % 6][v]);
            load(k + 3, w[(r + 5) % 6]);
            // output operands of point k-1, loaded before the arithmetic
            const size_t o = base + (size_t)(i >= 2 ? k - 1 : j0) * sg.lstride;
            const uint32_t bo = (uint32_t)(o * sizeof(T)), boa = (uint32_t)(o * sizeof(double));
            T pr[5], pu[5];
            double pa[5];
            if (i >= 2) {
                if constexpr (VISC) {  // the viscous term of the point joins the writing sweep
                    static_assert(DIR == 0 && MODE == MODE_WRITE, "the x sweep takes the viscous term");
#pragma unroll
                    for (int c = 0; c < 4; ++c) pr[1 + c] = __builtin_nontemporal_load(elem(vd, n3, c, bo));
                }
                if constexpr (MODE == MODE_ACCUM || is_rk(MODE)) {
#pragma unroll
                    for (int v = 0; v < 5; ++v) {
                        if constexpr (is_rk(MODE)) pr[v] = __builtin_nontemporal_load(elem(rhs_in, n3, v, bo));
                        else pr[v] = *elem(rhs_in, n3, v, bo);
                    }
                }
                if constexpr (MODE == MODE_RK2 || MODE == MODE_RK3) {
#pragma unroll
                    for (int v = 0; v < 5; ++v) pu[v] = *elem(un, n3, v, bo);
                }
                if constexpr (MODE == MODE_RK3) {
#pragma unroll
                    for (int v = 0; v < 5; ++v) pa[v] = __builtin_nontemporal_load(elem(acc, n3, v, boa));
                }
            }
            put_flux(r + 4, w[(r + 4) % 6]);
            const RoeCell<T> cb = roe_cell(w[(r + 2) % 6], gm1);
            // the fence between scalars keeps the scheduler from hoisting all the LDS
            // reads, which would hold them in registers across the reconstructions
            T du[5], Fs[5];
#pragma unroll
            for (int c = 0; c < kNS; ++c) {
                T s[5], lf, rf;
#pragma unroll
                for (int m = 0; m < 5; ++m) s[m] = c < 5 ? w[(r + m) % 6][c] : slot(r + m)[(c - 5) * 64];
                weno5_cell6<WW>(s[0], s[1], s[2], s[3], s[4], eps4, lf, rf);
                face_pair<T, DIR>(c, Lf[c], rf, du, Fs);
                Lf[c] = lf;
                pin(Lf[c]);
                __builtin_amdgcn_sched_barrier(0);
            }
            {
                T H[5];
                interface_flux<T, DIR>(du, Fs, ca, cb, gm1, delta, H);  // (unused at i = 0)
                if (i >= 2) {
#pragma unroll
                    for (int v = 0; v < 5; ++v) {
                        const T dH = Hp[v] - H[v];
                        if constexpr (is_rk(MODE)) {
                            // the stage state at the point: u^n itself in the first stage
                            rk_update<MODE>(L, dt, double(fmadd(dH, inv_dx, pr[v])), double(w[(r + 1) % 6][v]),
                                            MODE == MODE_RK1 ? 0.0 : double(pu[v]), MODE == MODE_RK3 ? pa[v] : 0.0,
                                            elem(unext, n3, v, bo), elem(acc, n3, v, boa));
                        } else if constexpr (MODE == MODE_ACCUM) {
                            *elem(rhs_out, n3, v, bo) = fmadd(dH, inv_dx, pr[v]);
                        } else if constexpr (MODE == MODE_RAW) {
                            *elem(rhs_out, n3, v, bo) = dH;
                        } else {
                            *elem(rhs_out, n3, v, bo) = VISC && v > 0 ? fmadd(dH, inv_dx, pr[v]) : dH * inv_dx;
                        }
                    }
                }
#pragma unroll
                for (int v = 0; v < 5; ++v) Hp[v] = H[v];
            }
            ca = cb;
        };
        for (int i = 0;;) {
            step(std::integral_constant<int, 0>{}, i);
            if (++i > len + 1) break;
            step(std::integral_constant<int, 1>{}, i);
            if (++i > len + 1) break;
            step(std::integral_constant<int, 2>{}, i);
            if (++i > len + 1) break;
#pragma unroll
            for (int m = 0; m < 3; ++m)
#pragma unroll
                for (int v = 0; v < 5; ++v) {
                    const T tmp = w[m][v];
                    w[m][v] = w[m + 3][v];
                    w[m + 3][v] = tmp;
                }
            T *const tmp = rlo;
            rlo = rhi;
            rhi = tmp;
        }
    }
}

template <typename T, int DIR, int MODE, bool VISC, int WW>
__global__ __launch_bounds__(256, 2) void k_sweep(Launch L0) {
    extern __shared__ unsigned char lds_raw[];
    const Launch L = with_params(L0);
    sweep_blocks<T, DIR, MODE, VISC, WW>(L, vb_range(L.total), lds_raw);
}

// ----------------------------------------------------------------------------
// x sweep: rows staged in LDS, lanes along x, two neighbouring cells per thread.
//
// A thread forms the face values of its cells A = 2s and B = 2s+1 from six staged points
// (the indicator terms of the stencils the cells share are formed once, and each staged
// value is read 3 times instead of 5), the flux at the face between them, then, with B's
// right-face values of its left neighbour, the flux at A's left face; the flux at B's
// right face comes from the right neighbour.  Against one cell per thread that halves the
// exchanges through LDS and the barriers per cell.  512^3: 5.43 -> 4.06 ms, 1044 -> 742 VALU
// instructions per point, 0.77 of the issue slots at the clock of the run (one cell per
// thread 6.4 ms, 834 instructions, waiting on LDS and barriers); 128^3: 0.106 -> 0.081 ms.
//
// Staged per point: the state, the velocity along x and the pressure (7 fields), from
// which the fluxes are formed as they are read; two ghost points on the left of a row and
// two or three on its right carry the periodic wrap.
// ----------------------------------------------------------------------------
template <typename T>
using vec2 = T __attribute__((ext_vector_type(2)));
constexpr int kXF = 7;                      // staged fields
constexpr int kXMax = 2 * kRowThreads;      // cells per block
// staged points of a row: its cells (rounded up to even), two ghosts on either side
__host__ __device__ __forceinline__ int xrow_points(int nx) { return (nx + 1) / 2 * 2 + 4; }
constexpr int kXPer = kXMax + 4;            // staged points of a chunk of a long row

template <typename T>
__device__ __forceinline__ void stage_point(T *st, int per, int pos, const T w[5], T vn, T p) {
#pragma unroll
    for (int v = 0; v < 5; ++v) st[v * per + pos] = w[v];
    st[5 * per + pos] = vn;
    st[6 * per + pos] = p;
}
template <typename T>
__device__ __forceinline__ void x_vel_pressure(const T w[5], T gm1, T &vn, T &p) {
#pragma clang fp contract(off)
    const T inv = rcp(w[0]);
    vn = w[1] * inv;
    p = gm1 * fmadd(T(-0.5), fmadd(w[1], vn, fmadd(w[2], w[2] * inv, w[3] * (w[3] * inv))), w[4]);
}

// Face values of the two cells whose six stencil points are staged from position `at`
// (even), one scalar at a time behind a scheduling fence, so that a reconstruction holds
// only the operands of the scalar in flight.  ar: A at its left face; du, Fs: the jumps
// and flux sums of the face between A and B; the right-face values of B (of A when there
// is no B) go to ex for the right neighbour.
template <typename T, int WW>
__device__ __forceinline__ void pair_faces(const T *st, int per, int at, T eps4, bool has_b, T *ex, T ar[kNS], T du[5],
                                           T Fs[5]) {
#pragma clang fp contract(off)
    auto get = [&](int f, T q[6]) {
        const vec2<T> *p = reinterpret_cast<const vec2<T> *>(st + f * per + at);
#pragma unroll
        for (int m = 0; m < 3; ++m) {
            const vec2<T> x = p[m];
            q[2 * m] = x.x;
            q[2 * m + 1] = x.y;
        }
    };
    T vn[6];
#pragma unroll
    for (int c = 0; c < kNS; ++c) {
        T q[6];
        get(c < 5 ? c : c - 4, q);
        if (c == 5) get(5, vn);
        if (c == 5 || c == 8) {
            T p[6];
            get(6, p);
#pragma unroll
            for (int m = 0; m < 6; ++m) q[m] = c == 5 ? fmadd(q[m], vn[m], p[m]) : (q[m] + p[m]) * vn[m];
        } else if (c > 5) {
#pragma unroll
            for (int m = 0; m < 6; ++m) q[m] = q[m] * vn[m];
        }
        T al, bl, br;
        weno5_cell6<WW>(q[0], q[1], q[2], q[3], q[4], eps4, al, ar[c]);
        weno5_cell6<WW>(q[1], q[2], q[3], q[4], q[5], eps4, bl, br);
        face_pair<T, 0>(c, al, br, du, Fs);
        ex[c * kRowThreads] = has_b ? bl : al;
        pin(ar[c]);
        __builtin_amdgcn_sched_barrier(0);
    }
}
template <typename T>
__device__ __forceinline__ RoeCell<T> staged_cell(const T *st, int per, int pos, T gm1) {
    T w[5];
#pragma unroll
    for (int v = 0; v < 5; ++v) w[v] = st[v * per + pos];
    return roe_cell(w, gm1);
}

// outputs at the two cells of a pair, o = offset of A: fluxes at A's left face, between
// the cells and at B's right face
template <typename T, bool VISC, bool RAW>
__device__ __forceinline__ void write_pair(gptr<T> out, gptr<const T> vd, size_t n3, size_t o, bool vec, bool has_b,
                                           const T Hl[5], const T Hi[5], const T Hn[5], T inv_dx) {
#pragma clang fp contract(off)
    T a[5], b[5], pa[4], pb[4];
    if constexpr (VISC) {
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            if (vec) {
                const vec2<T> x = __builtin_nontemporal_load((gptr<const vec2<T>>)(vd + c * n3 + o));
                pa[c] = x.x;
                pb[c] = x.y;
            } else {
                pa[c] = __builtin_nontemporal_load(vd + c * n3 + o);
                pb[c] = has_b ? __builtin_nontemporal_load(vd + c * n3 + o + 1) : T(0);
            }
        }
    }
#pragma unroll
    for (int v = 0; v < 5; ++v) {
        const T da = Hl[v] - Hi[v], db = Hi[v] - Hn[v];
        a[v] = RAW ? da : (VISC && v > 0 ? fmadd(da, inv_dx, pa[v - 1]) : da * inv_dx);
        b[v] = RAW ? db : (VISC && v > 0 ? fmadd(db, inv_dx, pb[v - 1]) : db * inv_dx);
        if (vec) {
            *(gptr<vec2<T>>)(out + v * n3 + o) = vec2<T>{a[v], b[v]};
        } else {
            out[v * n3 + o] = a[v];
            if (has_b) out[v * n3 + o + 1] = b[v];
        }
    }
}

// whole rows of at most kXMax points, `rows` of them per block
template <typename T, bool VISC, bool RAW, int WW>
__device__ __forceinline__ void x_rows_blocks(const Launch &L, const VbRange R, unsigned char *lds_raw) {
#pragma clang fp contract(off)
    T *const ex = reinterpret_cast<T *>(lds_raw);  // [9][256] face values handed to the right neighbour
    T *const st = ex + kNS * kRowThreads;          // [7][per] staged points; later [5][256] left-face fluxes
    // A block walks over several row groups (grid stride); the global loads of the next
    // group are issued into registers before the arithmetic of the current one, so their
    // latency overlaps it.
    T pw[2][5];
    auto fetch = [&](long long vb) {
        const int bi = find_box(L.off, L.nbox, vb);
        const BoxDesc &bx = L.boxes[bi];
        const long long row0 = (vb - L.off[bi]) * bx.rows;
        const int nact = (int)min((long long)bx.rows, (long long)bx.ny * bx.nz - row0) * bx.nx;
        const size_t n3 = uni64(bx.n3);
        const gptr<const T> u = uni(glob((const T *)state_ptr(bx, L, L.in)));
#pragma unroll
        for (int k = 0; k < 2; ++k) {
            const int m = threadIdx.x + k * kRowThreads;
            if (m < nact) {
                const uint32_t bo = (uint32_t)(((size_t)row0 * bx.nx + m) * sizeof(T));
#pragma unroll
                for (int v = 0; v < 5; ++v) pw[k][v] = *elem(u, n3, v, bo);
            }
        }
    };
    const int t = threadIdx.x;
    if (R.vb < R.end) fetch(R.vb);
    for (long long vb = R.vb; vb < R.end; vb += R.stride) {
        const int bi = find_box(L.off, L.nbox, vb);
        const BoxDesc &bx = L.boxes[bi];
        const int nx = bx.nx, hp = (nx + 1) / 2, rs = xrow_points(nx), per = bx.rows * rs;
        const size_t n3 = uni64(bx.n3);
        const T eps4 = T(4.0 * bx.eps), delta = T(bx.delta);
        const T gm1 = T(bx.gamma) - T(1);
        const T inv_dx = T(bx.inv_h[0]);
        const long long row0 = (vb - L.off[bi]) * bx.rows;
        const int nrow = (int)min((long long)bx.rows, (long long)bx.ny * bx.nz - row0);
        const gptr<T> out = uni(glob((T *)(L.out_ov && !RAW ? L.out_ov : bx.rhs)));
        const gptr<const T> vd = uni(glob((const T *)bx.G));
        // quotients of numbers below 2^16 by nx and hp: the rounding of the reciprocal moves
        // (m + 1/2) / n by less than its distance to the next integer
        const float inx = 1.0f / (float)nx, ihp = 1.0f / (float)hp;
#pragma unroll
        for (int k = 0; k < 2; ++k) {
            const int m = t + k * kRowThreads;
            if (m < nrow * nx) {
                const int r = (int)(((float)m + 0.5f) * inx), c = m - r * nx, pos = r * rs + 2 + c;
                T vn, p;
                x_vel_pressure(pw[k], gm1, vn, p);
                stage_point(st, per, pos, pw[k], vn, p);
                if (c <= 2 * hp + 1 - nx) stage_point(st, per, pos + nx, pw[k], vn, p);
                if (c >= nx - 2) stage_point(st, per, pos - nx, pw[k], vn, p);
            }
        }
        __syncthreads();
        if (vb + R.stride < R.end) fetch(vb + R.stride);
        const int r = (int)(((float)t + 0.5f) * ihp), s = t - r * hp;
        const bool act = r < nrow, has_b = 2 * s + 1 < nx;
        T ar[kNS], Hl[5], Hi[5];
        RoeCell<T> ca, cb;
        if (act) {
            const int at = r * rs + 2 * s;
            T du[5], Fs[5];
            pair_faces<T, WW>(st, per, at, eps4, has_b, ex + t, ar, du, Fs);
            cb = staged_cell(st, per, at + 2, gm1);
            interface_flux<T, 0>(du, Fs, cb, staged_cell(st, per, at + 3, gm1), gm1, delta, Hi);
#pragma unroll
            for (int v = 0; v < 5; ++v) pin(Hi[v]);
            ca = staged_cell(st, per, at + 1, gm1);
        }
        __syncthreads();  // the exchanged values are in place, every thread has read the staging
        if (act) {
            T du[5], Fs[5];
            const T *const el = ex + (s > 0 ? t - 1 : t + hp - 1);
#pragma unroll
            for (int c = 0; c < kNS; ++c) face_pair<T, 0>(c, el[c * kRowThreads], ar[c], du, Fs);
            interface_flux<T, 0>(du, Fs, ca, cb, gm1, delta, Hl);
#pragma unroll
            for (int v = 0; v < 5; ++v) st[v * kRowThreads + t] = Hl[v];
        }
        __syncthreads();
        if (act) {
            T Hn[5];
            const T *const hn = st + (s < hp - 1 ? t + 1 : t - (hp - 1));
#pragma unroll
            for (int v = 0; v < 5; ++v) Hn[v] = hn[v * kRowThreads];
            write_pair<T, VISC, RAW>(out, vd, n3, (size_t)(row0 + r) * nx + 2 * s, !(nx & 1), has_b, Hl, Hi, Hn, inv_dx);
        }
        __syncthreads();  // LDS is reused by the next virtual block
    }
}

template <typename T, bool VISC, int WW>
__global__ __launch_bounds__(kRowThreads, 2) void k_sweep_x_rows(Launch L0) {
    extern __shared__ unsigned char lds_raw[];
    const Launch L = with_params(L0);
    x_rows_blocks<T, VISC, false, WW>(L, vb_range(L.total), lds_raw);
}

// ----------------------------------------------------------------------------
// A stage of a small box (or of a few) in two launches: the viscous terms and the three
// sweeps side by side, each into a buffer of its own, then the sum of the four and the
// update point by point.  The sums take the terms in the order, and with the roundings,
// of the sweeps one after the other, so the results are the same bits.
//
// One after the other, small boxes pay four short kernels, each a fraction of the chip and as
// long as its chain of planes or cells (32^3: 17 + 8 + 9 + 10 us); side by side a stage takes
// the longest (32^3: 18 us) and 4.5 us for the sum.  At 64^3 the kernels share the chip: 46 us
// and 12 us for the sum's 24-34 fields, against 75.
// ----------------------------------------------------------------------------
struct SmallFams {
    const long long *off[4];  // viscous terms, z, y, x rows: prefixes and virtual blocks
    long long total[4];
};
template <bool VISC, bool DIAG, int WW>
__global__ __launch_bounds__(256, 2) void k_small(Launch L0, SmallFams F) {
    extern __shared__ unsigned char lds_raw[];
    Launch L = with_params(L0);
    long long b = blockIdx.x;
    int f = 0;
    while (f < 3 && b >= F.total[f]) b -= F.total[f++];
    L.off = F.off[f];
    L.total = F.total[f];
    const VbRange R{b, b + 1, 1};
    if (f == 0) {
        if constexpr (VISC) visc_blocks<double, DIAG>(L, R, *reinterpret_cast<ViscLds<double, DIAG> *>(lds_raw));
    } else if (f == 1) {
        sweep_blocks<double, 2, MODE_RAW, false, WW>(L, R, lds_raw);
    } else if (f == 2) {
        sweep_blocks<double, 1, MODE_RAW, false, WW>(L, R, lds_raw);
    } else {
        x_rows_blocks<double, false, true, WW>(L, R, lds_raw);
    }
}

template <int MODE, bool VISC>
__global__ __launch_bounds__(kPointThreads) void k_stage_sum(Launch L0) {
#pragma clang fp contract(off)
    const Launch L = with_params(L0);
    const long long vb = blockIdx.x;
    const int bi = find_box(L.off, L.nbox, vb);
    const BoxDesc &b = L.boxes[bi];
    const size_t n3 = uni64(b.n3), i = (size_t)(vb - L.off[bi]) * kPointThreads + threadIdx.x;
    if (i >= n3) return;
    const uint32_t bo = (uint32_t)(i * sizeof(double));
    const gptr<const double> dx = uni(raw_buf<double, 0>(b, L)), dy = uni(raw_buf<double, 1>(b, L)),
                             dz = uni(raw_buf<double, 2>(b, L)), vd = uni(glob((const double *)b.G));
    const gptr<const double> us = uni(glob((const double *)state_ptr(b, L, L.in))),
                             un = uni(glob((const double *)state_ptr(b, L, BUF_U)));
    const gptr<double> acc = uni(glob(b.acc)), unext = uni(glob((double *)state_ptr(b, L, L.out)));
    const gptr<double> rhs = uni(glob((double *)(L.out_ov ? L.out_ov : b.rhs)));
    const double ihx = b.inv_h[0], ihy = b.inv_h[1], ihz = b.inv_h[2];
    const double dt = L.dt_ov > 0.0 ? L.dt_ov : b.dt;
    double x[5], y[5], z[5], w[5], s[5], o[5], a[5];
#pragma unroll
    for (int v = 0; v < 5; ++v) {
        x[v] = *elem(dx, n3, v, bo), y[v] = *elem(dy, n3, v, bo), z[v] = *elem(dz, n3, v, bo);
        w[v] = VISC && v > 0 ? *elem(vd, n3, v - 1, bo) : 0.0;
        if constexpr (is_rk(MODE)) s[v] = *elem(us, n3, v, bo);
        o[v] = MODE == MODE_RK2 || MODE == MODE_RK3 ? *elem(un, n3, v, bo) : 0.0;
        a[v] = MODE == MODE_RK3 ? *elem(acc, n3, v, bo) : 0.0;
    }
#pragma unroll
    for (int v = 0; v < 5; ++v) {
        const double r = VISC && v > 0 ? fmadd(x[v], ihx, w[v]) : x[v] * ihx;
        const double kk = fmadd(z[v], ihz, fmadd(y[v], ihy, r));
        if constexpr (is_rk(MODE)) rk_update<MODE>(L, dt, kk, s[v], o[v], a[v], elem(unext, n3, v, bo), elem(acc, n3, v, bo));
        else *elem(rhs, n3, v, bo) = kk;
    }
}

// Rows longer than kXMax: one block walks one periodic row in chunks of kXMax cells, each
// staged with its ghost points.  A chunk's last cell waits for the next chunk, whose first
// thread finishes it (the cell's right-face values and left-face flux are carried in
// LDS); the row's first face waits for the last chunk.
constexpr int kCarry = kNS + 5;           // of a chunk's last cell: right-face values, left-face flux
constexpr int kFirst = kNS + 5 + 5 + 5;   // of the row's first cell: left-face values, right-face flux, Roe quantities of
                                          // the cells on either side of its left face
__host__ __device__ __forceinline__ size_t chunk_lds_bytes(size_t esz) {
    return (kNS * kRowThreads + kXF * kXPer + 2 * kCarry + kFirst) * esz;
}
__host__ __device__ __forceinline__ size_t rows_lds_bytes(int nx, int rows, size_t esz) {
    // the left-face fluxes reuse the staging
    return (kNS * kRowThreads + std::max(kXF * rows * xrow_points(nx), 5 * kRowThreads)) * esz;
}

template <typename T, bool VISC, int WW>
__global__ __launch_bounds__(kRowThreads, 2) void k_sweep_x_chunks(Launch L0) {
#pragma clang fp contract(off)
    const Launch L = with_params(L0);
    extern __shared__ unsigned char lds_raw[];
    T *const ex = reinterpret_cast<T *>(lds_raw);
    T *const st = ex + kNS * kRowThreads;
    T *const carry = st + kXF * kXPer;      // [2][kCarry], by chunk parity
    T *const first = carry + 2 * kCarry;    // [kFirst]
    const int t = threadIdx.x;
    auto put_cell = [&](T *d, const RoeCell<T> &c) { d[0] = c.s, d[1] = c.v[0], d[2] = c.v[1], d[3] = c.v[2], d[4] = c.H; };
    auto get_cell = [&](const T *d) { return RoeCell<T>{d[0], {d[1], d[2], d[3]}, d[4]}; };
    const VbRange R = vb_range(L.total);
    for (long long vb = R.vb; vb < R.end; vb += R.stride) {
        const int bi = find_box(L.off, L.nbox, vb);
        const BoxDesc &bx = L.boxes[bi];
        const int nx = bx.nx;
        const size_t n3 = uni64(bx.n3), obase = (size_t)(vb - L.off[bi]) * nx;
        const gptr<const T> u = uni(glob((const T *)state_ptr(bx, L, L.in)));
        const gptr<const T> vd = uni(glob((const T *)bx.G));
        const gptr<T> out = uni(glob((T *)(L.out_ov ? L.out_ov : bx.rhs)));
        const T eps4 = T(4.0 * bx.eps), delta = T(bx.delta);
        const T gm1 = T(bx.gamma) - T(1);
        const T inv_dx = T(bx.inv_h[0]);
        const int nch = (nx + kXMax - 1) / kXMax;
        // the point of one cell from the fluxes of its faces
        auto write_cell = [&](int i, const T *Ha, const T Hb[5]) {
            const size_t o = obase + i;
#pragma unroll
            for (int v = 0; v < 5; ++v) {
                const T dH = Ha[v] - Hb[v];
                out[v * n3 + o] = VISC && v > 0 ? fmadd(dH, inv_dx, vd[(v - 1) * n3 + o]) : dH * inv_dx;
            }
        };
        for (int c = 0; c < nch; ++c) {
            const int i0 = c * kXMax, cells = min(kXMax, nx - i0);
            for (int sp = t; sp < cells + 4 + (cells & 1); sp += kRowThreads) {
                const size_t o = obase + wrapm(i0 - 2 + sp, nx);
                T w[5], vn, p;
#pragma unroll
                for (int v = 0; v < 5; ++v) w[v] = u[v * n3 + o];
                x_vel_pressure(w, gm1, vn, p);
                stage_point(st, kXPer, sp, w, vn, p);
            }
            __syncthreads();
            const int i = i0 + 2 * t;  // cell A
            const bool act = 2 * t < cells, has_b = 2 * t + 1 < cells, last = 2 * t + 2 >= cells;
            T *const cn = carry + (c & 1) * kCarry, *const cp = carry + (~c & 1) * kCarry;
            T ar[kNS], Hl[5], Hi[5];
            RoeCell<T> ca, cb;
            if (act) {
                T du[5], Fs[5];
                pair_faces<T, WW>(st, kXPer, 2 * t, eps4, has_b, ex + t, ar, du, Fs);
                cb = staged_cell(st, kXPer, 2 * t + 2, gm1);
                interface_flux<T, 0>(du, Fs, cb, staged_cell(st, kXPer, 2 * t + 3, gm1), gm1, delta, Hi);
#pragma unroll
                for (int v = 0; v < 5; ++v) pin(Hi[v]);
                ca = staged_cell(st, kXPer, 2 * t + 1, gm1);
                if (i == 0) {
#pragma unroll
                    for (int s = 0; s < kNS; ++s) first[s] = ar[s];
#pragma unroll
                    for (int v = 0; v < 5; ++v) first[kNS + v] = Hi[v];
                    put_cell(first + kNS + 5, ca);
                    put_cell(first + kNS + 10, cb);
                }
            }
            __syncthreads();  // the exchanged values are in place, every thread has read the staging
            if (t < kNS) cn[t] = ex[t * kRowThreads + (cells + 1) / 2 - 1];
            if (act && i > 0) {
                T du[5], Fs[5];
#pragma unroll
                for (int s = 0; s < kNS; ++s)
                    face_pair<T, 0>(s, t > 0 ? ex[s * kRowThreads + t - 1] : cp[s], ar[s], du, Fs);
                interface_flux<T, 0>(du, Fs, ca, cb, gm1, delta, Hl);
#pragma unroll
                for (int v = 0; v < 5; ++v) st[v * kRowThreads + t] = Hl[v];
            }
            if (act && last)
#pragma unroll
                for (int v = 0; v < 5; ++v) cn[kNS + v] = has_b ? Hi[v] : Hl[v];
            __syncthreads();
            // the chunk's last cell waits for the next chunk, whose first thread finishes it
            if (act && !last) {
                T Hn[5];
#pragma unroll
                for (int v = 0; v < 5; ++v) Hn[v] = st[v * kRowThreads + t + 1];
                if (i > 0) write_pair<T, VISC, false>(out, vd, n3, obase + i, !(nx & 1), true, Hl, Hi, Hn, inv_dx);
                else write_cell(1, Hi, Hn);
            } else if (act && has_b && i > 0) {
                write_cell(i, Hl, Hi);
            }
            if (t == 0 && c > 0) write_cell(i0 - 1, cp + kNS, Hl);
            __syncthreads();  // the next chunk overwrites the staging
        }
        if (t == 0) {
            // the face at the row's wrap, its first and its last point
            const T *const cl = carry + ((nch - 1) & 1) * kCarry;
            T du[5], Fs[5], H[5], Hr[5];
#pragma unroll
            for (int s = 0; s < kNS; ++s) face_pair<T, 0>(s, cl[s], first[s], du, Fs);
            interface_flux<T, 0>(du, Fs, get_cell(first + kNS + 5), get_cell(first + kNS + 10), gm1, delta, H);
#pragma unroll
            for (int v = 0; v < 5; ++v) Hr[v] = first[kNS + v];
            write_cell(nx - 1, cl + kNS, H);
            write_cell(0, H, Hr);
        }
        __syncthreads();  // LDS is reused by the next row
    }
}

// ----------------------------------------------------------------------------
// diagnostics: deterministic two-pass reduction per box
// ----------------------------------------------------------------------------
__device__ __forceinline__ double wave_sum(double v) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
    return v;
}
__device__ __forceinline__ double wave_max(double v) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v = fmax(v, __shfl_xor(v, o, 64));
    return v;
}
// the diagnostics walk the box in the tiles of the viscous-flux kernel (32 x 8 columns,
// diag_planes planes); one partial-sum block per tile, at most kDiagBlocksMax (then a
// block takes every kDiagBlocksMax-th tile)
__host__ __device__ __forceinline__ int diag_blocks(int nx, int ny, int nz) {
    const long long t = diag_tiles(nx, ny, nz);
    return (int)(t < kDiagBlocksMax ? t : kDiagBlocksMax);
}

// block reduction over NW waves of CNS_NDIAG values (slot 7 a max, the others sums) in a
// fixed order: those of `mask` are reduced and written to dst
template <int NW>
__device__ __forceinline__ void block_reduce_diag(const double acc[CNS_NDIAG], double (*red)[CNS_NDIAG],
                                                  gptr<double> dst, unsigned mask) {
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
#pragma unroll
    for (int d = 0; d < CNS_NDIAG; ++d) {
        if (!(mask >> d & 1)) continue;
        double v = (d == 7) ? wave_max(acc[d]) : wave_sum(acc[d]);
        if (lane == 0) red[wid][d] = v;
    }
    __syncthreads();
    if (threadIdx.x < CNS_NDIAG && (mask >> threadIdx.x & 1)) {
        const int d = threadIdx.x;
        double v = red[0][d];
        for (int w2 = 1; w2 < NW; ++w2) v = (d == 7) ? fmax(v, red[w2][d]) : v + red[w2][d];
        if (dst) dst[d] = v;
    }
    __syncthreads();
}

static_assert(kDiagThreads == kViscTX * kViscTY, "one thread to each column of a kViscTX x kViscTY tile");

// velocity m/rho of a state
__device__ __forceinline__ void vel_of(const double s[5], double v[3]) {
#pragma clang fp contract(off)
    const double ir = rcp(s[0]);
    v[0] = s[1] * ir;
    v[1] = s[2] * ir;
    v[2] = s[3] * ir;
}

// The point quantities and sums of a record state every operation (contraction off), here, in
// the kernels below and in the viscous kernel (prim_stats), so that a record has the same bits
// from every kernel and variant that forms it.

// Point quantities of one state (kinetic energy, mass, momentum, energy, the largest
// wave speed |v_d| + c, the bad-point count) added to acc; returns whether the point is
// valid (finite, rho > 0, p > 0) and its velocity in v.
__device__ __forceinline__ bool point_stats(const double s[5], double gamma, double acc[CNS_NDIAG], double v[3]) {
#pragma clang fp contract(off)
    const double r = s[0], mx = s[1], my = s[2], mz = s[3], e = s[4];
    const double inv = rcp(r);
    v[0] = mx * inv;
    v[1] = my * inv;
    v[2] = mz * inv;
    const double ke = 0.5 * fma(mz, v[2], fma(my, v[1], mx * v[0]));
    const double p = (gamma - 1.0) * (e - ke);
    const bool finite = isfinite(r) && isfinite(mx) && isfinite(my) && isfinite(mz) && isfinite(e);
    if (!finite || !(r > 0.0) || !(p > 0.0)) {
        acc[8] += 1.0;
        return false;
    }
    acc[0] += ke;
    acc[2] += r;
    acc[3] += mx;
    acc[4] += my;
    acc[5] += mz;
    acc[6] += e;
    const double c = sqrt(gamma * p * inv);
    acc[7] = fmax(acc[7], fmax(fabs(v[0]), fmax(fabs(v[1]), fabs(v[2]))) + c);
    return true;
}

// Per-block partial diagnostics on the tiles of the viscous-flux kernel.  Each state
// value is loaded once per tile: a thread loads its column at plane k+2 (the point
// quantities of that plane are summed then, in plane order) and, if it owns a point of
// the halo ring, that point at plane k+2 as well; the vorticity of plane k takes the
// 4th-order central derivative of the velocity, whose x and y neighbours come from an
// LDS copy of plane k staged from the column and ring windows, and whose z neighbours
// from the column's window of five planes in registers.  The loads of a plane are issued
// a plane ahead of its use: 128^3 34.8 -> 29.4 us, in the mixed form at 256^3 171 -> 134.  In a
// large FP64 box (512^3 1.6 ms as before) the rate of the caches at which the tiles' 1.5 times the
// state with halos come bounds it.  OCC, blocks on a CU: four hold all 1024 blocks of such a box
// at once (with three 512^3 took 1.72 ms); where three suffice, FP64 takes the variant without
// spills (128^3: 31.6 us with four).
template <typename T, int OCC>
__global__ __launch_bounds__(kDiagThreads, OCC) void k_diag_partial(Launch L0) {
#pragma clang fp contract(off)
    const Launch L = with_params(L0);
    __shared__ double red[kDiagThreads / 64][CNS_NDIAG];
    __shared__ double pv[3][kViscTY + 4][kViscTX + 4];
    __shared__ double rv[3][3][kViscRing];  // ring velocities, slot (plane - z0) mod 3
    int rhx, rhy;
    ring_pos(threadIdx.x, rhx, rhy);
    const bool ring = threadIdx.x < kViscRing;
    const int rt = ring ? threadIdx.x : 0;
    const VbRange R = vb_range(L.total);
    for (long long vb = R.vb; vb < R.end; vb += R.stride) {
        const int bi = find_box(L.off, L.nbox, vb);
        const BoxDesc &bx = L.boxes[bi];
        const int nx = bx.nx, ny = bx.ny, nz = bx.nz;
        const size_t n3 = uni64(bx.n3), sz = (size_t)nx * ny;
        const int nblk = diag_blocks(nx, ny, nz);
        const long long ntile = diag_tiles(nx, ny, nz);
        const int grp = diag_planes(nx, ny, nz);
        const int lb = (int)(vb - L.off[bi]);
        const gptr<const T> u = uni(glob((const T *)state_ptr(bx, L, BUF_U)));
        const double gamma = bx.gamma;
        // the 1/12 of the central differences is folded into the spacings
        const double ihx = bx.inv_h[0] / 12.0, ihy = bx.inv_h[1] / 12.0, ihz = bx.inv_h[2] / 12.0;
        const int ntx = (nx + kViscTX - 1) / kViscTX, nty = (ny + kViscTY - 1) / kViscTY;
        const int tx = threadIdx.x % kViscTX, ty = threadIdx.x / kViscTX;
        double acc[CNS_NDIAG] = {0, 0, 0, 0, 0, 0, 0, 0, 0};
        for (long long tile = lb; tile < ntile; tile += nblk) {
            const int x0 = (int)(tile % ntx) * kViscTX, y0 = (int)((tile / ntx) % nty) * kViscTY;
            const int z0 = (int)(tile / ((long long)ntx * nty)) * grp, z1 = min(z0 + grp, nz);
            const bool act = x0 + tx < nx && y0 + ty < ny;
            // a column past a ragged edge wraps periodically (halo of the columns beside it)
            const uint32_t col = (uint32_t)wrapm(y0 + ty, ny) * nx + wrapm(x0 + tx, nx);
            const uint32_t rcol = (uint32_t)wrapm(y0 - 2 + rhy, ny) * nx + wrapm(x0 - 2 + rhx, nx);
            double vz[5][3];    // this column's velocity at planes k-2 .. k+2
            unsigned good = 0;  // bit m: the column's point at plane k-2+m is valid
            // the loads of plane k+2 (column and ring point) are issued a plane ahead
            T sn[5], rn[4];
            auto load_col = [&](int zp, T s[5]) {
                const uint32_t bo = (uint32_t)((col + wrapi(zp, nz) * sz) * sizeof(T));
#pragma unroll
                for (int c = 0; c < 5; ++c) s[c] = *elem(u, n3, c, bo);
            };
            auto load_ring = [&](int zp, T s[4]) {
                const uint32_t bo = (uint32_t)((rcol + wrapi(zp, nz) * sz) * sizeof(T));
#pragma unroll
                for (int c = 0; c < 4; ++c) s[c] = *elem(u, n3, c, bo);
            };
            // the four planes before them at once, or in two pairs where that would hold too much
            constexpr int H = sizeof(T) == 8 && OCC == 4 ? 2 : 4;
#pragma unroll
            for (int h = 0; h < 4; h += H) {
                T s4[H][5], r1[H / 2][4];
#pragma unroll
                for (int m = 0; m < H; ++m) load_col(z0 - 2 + h + m, s4[m]);
                if (ring)
#pragma unroll
                    for (int m = 0; m < H / 2; ++m) load_ring(z0 + h / 2 + m, r1[m]);
                if (h + H == 4) {
                    load_col(z0 + 2, sn);
                    if (ring) load_ring(z0 + 2, rn);
                }
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int m = 0; m < H; ++m) {
                    const int zp = z0 - 2 + h + m;
                    const double s[5] = {double(s4[m][0]), double(s4[m][1]), double(s4[m][2]), double(s4[m][3]),
                                         double(s4[m][4])};
                    if (act && zp >= z0 && zp < z1) {
                        if (point_stats(s, gamma, acc, vz[h + m])) good |= 1u << (h + m);
                    } else {
                        vel_of(s, vz[h + m]);
                    }
                }
                if (ring)
#pragma unroll
                    for (int m = 0; m < H / 2; ++m) {
                        const double ir = rcp(double(r1[m][0]));
#pragma unroll
                        for (int c = 0; c < 3; ++c) rv[h / 2 + m][c][rt] = double(r1[m][1 + c]) * ir;
                    }
            }
            int slot = 0;  // (k - z0) mod 3
            for (int k = z0; k < z1; ++k) {
                const int slot2 = slot == 0 ? 2 : slot - 1;  // (k + 2 - z0) mod 3
                const double s[5] = {double(sn[0]), double(sn[1]), double(sn[2]), double(sn[3]), double(sn[4])};
                const double r4[4] = {double(rn[0]), double(rn[1]), double(rn[2]), double(rn[3])};
                if (k + 1 < z1) {
                    load_col(k + 3, sn);
                    if (ring) load_ring(k + 3, rn);
                    __builtin_amdgcn_sched_barrier(0);
                }
                {
                    if (act && k + 2 < z1) {
                        if (point_stats(s, gamma, acc, vz[4])) good |= 1u << 4;
                    } else {
                        vel_of(s, vz[4]);
                    }
                }
                if (ring) {
                    const double ir = rcp(r4[0]);
#pragma unroll
                    for (int c = 0; c < 3; ++c) {
                        rv[slot2][c][rt] = r4[1 + c] * ir;
                        pv[c][rhy][rhx] = rv[slot][c][rt];
                    }
                }
#pragma unroll
                for (int c = 0; c < 3; ++c) pv[c][ty + 2][tx + 2] = vz[2][c];
                __syncthreads();
                if (act && (good & 4u)) {
                    // vorticity with the 4th-order central derivative
                    const int X = tx + 2, Y = ty + 2;
                    const double dvzdy = dcen12(pv[2][Y - 2][X], pv[2][Y - 1][X], pv[2][Y + 1][X], pv[2][Y + 2][X]) * ihy;
                    const double dvydz = dcen12(vz[0][1], vz[1][1], vz[3][1], vz[4][1]) * ihz;
                    const double dvxdz = dcen12(vz[0][0], vz[1][0], vz[3][0], vz[4][0]) * ihz;
                    const double dvzdx = dcen12(pv[2][Y][X - 2], pv[2][Y][X - 1], pv[2][Y][X + 1], pv[2][Y][X + 2]) * ihx;
                    const double dvydx = dcen12(pv[1][Y][X - 2], pv[1][Y][X - 1], pv[1][Y][X + 1], pv[1][Y][X + 2]) * ihx;
                    const double dvxdy = dcen12(pv[0][Y - 2][X], pv[0][Y - 1][X], pv[0][Y + 1][X], pv[0][Y + 2][X]) * ihy;
                    const double ox = dvzdy - dvydz, oy = dvxdz - dvzdx, oz = dvydx - dvxdy;
                    if (isfinite(ox) && isfinite(oy) && isfinite(oz)) acc[1] = fma(0.5, fma(oz, oz, fma(oy, oy, ox * ox)), acc[1]);
                }
                __syncthreads();  // the next plane overwrites the LDS tile
#pragma unroll
                for (int m = 0; m < 4; ++m)
#pragma unroll
                    for (int c = 0; c < 3; ++c) vz[m][c] = vz[m + 1][c];
                good >>= 1;
                slot = slot == 2 ? 0 : slot + 1;
            }
        }
        block_reduce_diag<kDiagThreads / 64>(acc, red, glob(bx.part) + (size_t)lb * CNS_NDIAG, ~0u);
    }
}

__global__ __launch_bounds__(kDiagThreads) void k_diag_final(Launch L0) {
    const Launch L = with_params(L0);
    __shared__ double red[kDiagThreads / 64][CNS_NDIAG];
    for (long long vb = blockIdx.x; vb < L.total; vb += gridDim.x) {
        const int bi = (int)vb;  // one virtual block per box
        const BoxDesc &bx = L.boxes[bi];
        const int nblk = L.diag_fused ? (int)diag_tiles(bx.nx, bx.ny, bx.nz) : diag_blocks(bx.nx, bx.ny, bx.nz);
        double acc[CNS_NDIAG] = {0, 0, 0, 0, 0, 0, 0, 0, 0};
        for (int b = threadIdx.x; b < nblk; b += kDiagThreads)
#pragma unroll
            for (int d = 0; d < CNS_NDIAG; ++d) {
                const double v = glob(bx.part)[(size_t)b * CNS_NDIAG + d];
                acc[d] = (d == 7) ? fmax(acc[d], v) : acc[d] + v;
            }
        const double inv = 1.0 / (double)bx.n3;
        const gptr<double> dst = L.diag ? glob(L.diag) + ((size_t)bi * L.diag_box_stride + L.step) * CNS_NDIAG : nullptr;
        block_reduce_diag<kDiagThreads / 64>(acc, red, dst, ~0u);
        // the thread that wrote a mean's sum divides it by the number of points
        if (dst && threadIdx.x < 7) dst[threadIdx.x] *= inv;
    }
}

// ----------------------------------------------------------------------------
// the CFL wave speed alone: max over points and directions of |v_d| + c (the same
// point arithmetic as slot 7 of the diagnostics), two passes per box
// ----------------------------------------------------------------------------
template <typename T>
__global__ __launch_bounds__(kDiagThreads) void k_speed_partial(Launch L0) {
#pragma clang fp contract(off)
    const Launch L = with_params(L0);
    __shared__ double red[kDiagThreads / 64][2];
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
    const VbRange R = vb_range(L.total);
    for (long long vb = R.vb; vb < R.end; vb += R.stride) {
        const int bi = find_box(L.off, L.nbox, vb);
        const BoxDesc &bx = L.boxes[bi];
        const int nblk = diag_blocks(bx.nx, bx.ny, bx.nz);
        const int lb = (int)(vb - L.off[bi]);
        const gptr<const T> u = glob((const T *)state_ptr(bx, L, BUF_U));
        const size_t n3 = bx.n3;
        const double gamma = bx.gamma;
        double smax = 0.0, bad = 0.0;
        for (size_t i = (size_t)lb * kDiagThreads + threadIdx.x; i < n3; i += (size_t)nblk * kDiagThreads) {
            const double r = double(u[i]), mx = double(u[n3 + i]), my = double(u[2 * n3 + i]),
                         mz = double(u[3 * n3 + i]), e = double(u[4 * n3 + i]);
            const double inv = rcp(r);
            const double vx = mx * inv, vy = my * inv, vzc = mz * inv;
            const double ke = 0.5 * fma(mz, vzc, fma(my, vy, mx * vx));
            const double p = (gamma - 1.0) * (e - ke);
            const bool finite = isfinite(r) && isfinite(mx) && isfinite(my) && isfinite(mz) && isfinite(e);
            if (!finite || !(r > 0.0) || !(p > 0.0)) {
                bad += 1.0;
            } else {
                const double c = sqrt(gamma * p * inv);
                smax = fmax(smax, fmax(fabs(vx), fmax(fabs(vy), fabs(vzc))) + c);
            }
        }
        smax = wave_max(smax);
        bad = wave_sum(bad);
        if (lane == 0) {
            red[wid][0] = smax;
            red[wid][1] = bad;
        }
        __syncthreads();
        if (threadIdx.x == 0) {
            double m = red[0][0], b = red[0][1];
            for (int w2 = 1; w2 < kDiagThreads / 64; ++w2) {
                m = fmax(m, red[w2][0]);
                b += red[w2][1];
            }
            glob(bx.part)[(size_t)lb * CNS_NDIAG + 7] = m;
            glob(bx.part)[(size_t)lb * CNS_NDIAG + 8] = b;
        }
        __syncthreads();
    }
}

__global__ __launch_bounds__(kDiagThreads) void k_speed_final(Launch L0, double *out) {
    const Launch L = with_params(L0);
    __shared__ double red[kDiagThreads / 64][2];
    for (long long vb = blockIdx.x; vb < L.total; vb += gridDim.x) {
        const int bi = (int)vb;  // one virtual block per box
        const BoxDesc &bx = L.boxes[bi];
        const int nblk = diag_blocks(bx.nx, bx.ny, bx.nz);
        double m = 0.0, b = 0.0;
        for (int k = threadIdx.x; k < nblk; k += kDiagThreads) {
            m = fmax(m, glob(bx.part)[(size_t)k * CNS_NDIAG + 7]);
            b += glob(bx.part)[(size_t)k * CNS_NDIAG + 8];
        }
        m = wave_max(m);
        b = wave_sum(b);
        if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6][0] = m, red[threadIdx.x >> 6][1] = b;
        __syncthreads();
        if (threadIdx.x == 0) {
            for (int w = 1; w < kDiagThreads / 64; ++w) m = fmax(m, red[w][0]), b += red[w][1];
            out[bi] = b > 0.0 ? __builtin_nan("") : m;
        }
        __syncthreads();
    }
}

// streaming copy of n16 16-byte words (bandwidth reference): each thread moves four
// words per round, the loads of a round issued before its stores
typedef double v2d __attribute__((ext_vector_type(2)));
__global__ __launch_bounds__(256) void k_stream_copy(const v2d *__restrict__ src, v2d *__restrict__ dst,
                                                     size_t n16) {
    const size_t stride = (size_t)gridDim.x * blockDim.x;
    size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    for (; i + 3 * stride < n16; i += 4 * stride) {
        v2d a = __builtin_nontemporal_load(&src[i]);
        v2d b = __builtin_nontemporal_load(&src[i + stride]);
        v2d c = __builtin_nontemporal_load(&src[i + 2 * stride]);
        v2d d = __builtin_nontemporal_load(&src[i + 3 * stride]);
        __builtin_nontemporal_store(a, &dst[i]);
        __builtin_nontemporal_store(b, &dst[i + stride]);
        __builtin_nontemporal_store(c, &dst[i + 2 * stride]);
        __builtin_nontemporal_store(d, &dst[i + 3 * stride]);
    }
    for (; i < n16; i += stride) __builtin_nontemporal_store(__builtin_nontemporal_load(&src[i]), &dst[i]);
}

__global__ void k_set_params(GraphParams *gp, const void *u, double *diag, double dt) {
    if (threadIdx.x == 0 && blockIdx.x == 0) {
        gp->u = u;
        gp->diag = diag;
        gp->dt = dt;
        gp->pad = 0.0;
    }
}

// ----------------------------------------------------------------------------
// host side: shapes, block counts, launchers
// ----------------------------------------------------------------------------
// as many rows as the pairs of a block's threads hold, the staging (7 fields) at most
// 34 KiB in FP64, which keeps three blocks on a CU
int rows_max(int nx) {
    return std::max(1, std::min(kRowThreads / ((nx + 1) / 2), 608 / xrow_points(nx)));
}

size_t xrows_lds(int nx, int rows, size_t esz) { return rows_lds_bytes(nx, rows, esz); }

// (the bound of the mixed form's kernel, four points per thread and its 14 staged fields; the FP64
// kernel takes what a caller sets within it down to rows_max)
bool rows_fit(int nx, int rows, size_t esz) {
    const long long per = (long long)rows * nx;
    return rows >= 1 && per <= 4 * kRowThreads && (size_t)14 * per * esz <= (size_t)kRowLdsMax;
}

long long family_blocks(const BoxDesc &b, int fam, int block) {
    switch (fam) {
        case F_POINT: return cdiv((long long)b.n3, kPointThreads);
        case F_XROWS: return b.xrows == 1 ? cdiv((long long)b.ny * b.nz, b.rows) : 0;
        case F_XCHUNK: return b.xrows == 2 ? (long long)b.ny * b.nz : 0;
        case F_SWEEP_X:
        case F_SWEEP_Y:
        case F_SWEEP_Z: {
            const int d = fam - F_SWEEP_X;
            if (d == 0 && b.xrows) return 0;
            const SweepGeom g = d == 0 ? sweep_geom<0>(b.nx, b.ny, b.nz)
                                       : (d == 1 ? sweep_geom<1>(b.nx, b.ny, b.nz) : sweep_geom<2>(b.nx, b.ny, b.nz));
            if (d == 1)  // blocks of 64 lines x (block/64) segments
                return cdiv(g.npq, 64) * cdiv(cdiv(g.nline, b.seg[d]), block / 64);
            return cdiv((long long)g.npq * cdiv(g.nline, b.seg[d]), block);
        }
        case F_DIAG: return diag_blocks(b.nx, b.ny, b.nz);
        case F_VISC: return plane_tiles(b.nx, b.ny, b.nz, b.vsz);
        case F_BOX: return 1;
    }
    return 0;
}

void launch_init_state(int prec, size_t n3, double gamma, const double *rho, const double *vel, const double *p,
                       void *u, hipStream_t s) {
    const unsigned g = (unsigned)((n3 + 255) / 256);
    if (prec == CNS_FP64)
        hipLaunchKernelGGL(k_init_state<double>, dim3(g), dim3(256), 0, s, n3, gamma - 1.0, rho, vel, p, (double *)u);
    else
        hipLaunchKernelGGL(k_init_state<float>, dim3(g), dim3(256), 0, s, n3, gamma - 1.0, rho, vel, p, (float *)u);
}

void launch_fill(int prec, size_t n, void *out, hipStream_t s) {
    const unsigned g = (unsigned)((n + 255) / 256);
    if (prec == CNS_FP64) hipLaunchKernelGGL(k_fill<double>, dim3(g), dim3(256), 0, s, n, (double *)out);
    else hipLaunchKernelGGL(k_fill<float>, dim3(g), dim3(256), 0, s, n, (float *)out);
}

// The launchers are templated on the state type: float hands over to the mixed form's own.
template <typename T>
constexpr bool kMixed = std::is_same<T, float>::value;

template <typename T, bool DIAG = false>
static void visc_fields(const Batch &bt, Launch L) {
    if constexpr (kMixed<T>) {
        mixed::visc_fields(bt, L);
    } else {
        L = with_family(bt, L, F_VISC);
        if (!L.total) return;
        ProfScope ps(bt.prof, K_VISC_FLUX, bt.stream);
        hipLaunchKernelGGL((k_visc<T, DIAG>), dim3(grid_of(bt, F_VISC, L.total)),
                           dim3(ViscTile<T>::kThreads), 0, bt.stream,
                           L);
    }
}

// flux ring of the marching sweeps: 6 slots x 4 per thread
static size_t sweep_lds_bytes(int block) { return 24 * (size_t)block * sizeof(double); }

template <typename T, int DIR, int MODE, bool VISC>
static void sweep_t(const Batch &bt, const Launch &L) {
    const dim3 g(grid_of(bt, F_SWEEP_X + DIR, L.total)), b(bt.block);
    const size_t ring = sweep_lds_bytes(bt.block);
    if (bt.weights == CNS_WENO_Z)
        hipLaunchKernelGGL((k_sweep<T, DIR, MODE, VISC, CNS_WENO_Z>), g, b, ring, bt.stream, L);
    else if (bt.weights == CNS_WENO_M)
        hipLaunchKernelGGL((k_sweep<T, DIR, MODE, VISC, CNS_WENO_M>), g, b, ring, bt.stream, L);
    else
        hipLaunchKernelGGL((k_sweep<T, DIR, MODE, VISC, CNS_WENO_JS>), g, b, ring, bt.stream, L);
}

template <typename T, int MODE>
static void sweep(const Batch &bt, Launch L, int dir, bool visc) {
    if constexpr (kMixed<T>) {
        if constexpr (MODE == MODE_WRITE) mixed::sweep_write(bt, L, dir, visc);
        else mixed::sweep_accum(bt, L, dir, visc);
    } else {
        L = with_family(bt, L, F_SWEEP_X + dir);
        if (!L.total) return;
        if (dir == 0) {  // the writing sweep, which takes the viscous term
            if constexpr (MODE == MODE_WRITE) {
                if (visc) sweep_t<T, 0, MODE, true>(bt, L);
                else sweep_t<T, 0, MODE, false>(bt, L);
            }
        } else if (dir == 1) {
            if constexpr (!is_rk(MODE)) sweep_t<T, 1, MODE, false>(bt, L);
        } else {
            sweep_t<T, 2, MODE, false>(bt, L);
        }
    }
}

// the z sweep with the fused update of stage L.stage of L.scheme
template <typename T>
static void sweep_rk(const Batch &bt, const Launch &L) {
    if constexpr (kMixed<T>) mixed::sweep_rk(bt, L, bt.any_visc);
    else if (L.stage == 1) sweep<T, MODE_RK1>(bt, L, 2, false);
    else if (L.scheme == CNS_RK4 && L.stage == 4) sweep<T, MODE_RK3>(bt, L, 2, false);
    else sweep<T, MODE_RK2>(bt, L, 2, false);
}

template <typename T, bool VISC, int WW>
static void xrows_tw(const Batch &bt, const Launch &L) {
    // about four row groups per block, so that the loads of the next one are prefetched
    const long long nb = bt.grid[F_XROWS] > 0 ? std::min<long long>(bt.grid[F_XROWS], L.total)
                                              : std::max<long long>(std::min<long long>(L.total, 2048), L.total / 4);
    hipLaunchKernelGGL((k_sweep_x_rows<T, VISC, WW>), dim3(grid_for(nb)), dim3(kRowThreads), bt.rowLds, bt.stream,
                       L);
}

template <typename T, bool VISC>
static void xrows_t(const Batch &bt, const Launch &L) {
    if (bt.weights == CNS_WENO_Z) xrows_tw<T, VISC, CNS_WENO_Z>(bt, L);
    else if (bt.weights == CNS_WENO_M) xrows_tw<T, VISC, CNS_WENO_M>(bt, L);
    else xrows_tw<T, VISC, CNS_WENO_JS>(bt, L);
}

template <typename T, bool VISC>
static void xchunks_t(const Batch &bt, const Launch &L) {
    const dim3 g(grid_of(bt, F_XCHUNK, L.total)), b(kRowThreads);
    const size_t lds = chunk_lds_bytes(sizeof(T));
    if (bt.weights == CNS_WENO_Z)
        hipLaunchKernelGGL((k_sweep_x_chunks<T, VISC, CNS_WENO_Z>), g, b, lds, bt.stream, L);
    else if (bt.weights == CNS_WENO_M)
        hipLaunchKernelGGL((k_sweep_x_chunks<T, VISC, CNS_WENO_M>), g, b, lds, bt.stream, L);
    else
        hipLaunchKernelGGL((k_sweep_x_chunks<T, VISC, CNS_WENO_JS>), g, b, lds, bt.stream, L);
}

// x sweep (always the first, writing sweep): the rows kernel for boxes whose rows fill at
// most one block, the chunked rows kernel for longer rows, the marching kernel when chosen
template <typename T>
static void sweep_x(const Batch &bt, const Launch &L, bool visc) {
    if constexpr (kMixed<T>) {
        mixed::sweep_x(bt, L, visc);
    } else {
        ProfScope ps(bt.prof, K_SWEEP_X, bt.stream);
        const Launch R = with_family(bt, L, F_XROWS);
        if (R.total) {
            if (visc) xrows_t<T, true>(bt, R);
            else xrows_t<T, false>(bt, R);
        }
        const Launch C = with_family(bt, L, F_XCHUNK);
        if (C.total) {
            if (visc) xchunks_t<T, true>(bt, C);
            else xchunks_t<T, false>(bt, C);
        }
        sweep<T, MODE_WRITE>(bt, L, 0, visc);
    }
}

// not while kernels are timed one by one (same bits either way)
static bool small_stage(const Batch &bt) { return bt.small && !(bt.prof && bt.prof->on); }

template <bool VISC, bool DIAG>
static void small_sweeps(const Batch &bt, const Launch &L) {
    SmallFams F{};
    const int fam[4] = {F_VISC, F_SWEEP_Z, F_SWEEP_Y, F_XROWS};
    long long total = 0;
    for (int k = VISC ? 0 : 1; k < 4; ++k) {
        F.off[k] = bt.d_off[fam[k]];
        F.total[k] = bt.total[fam[k]];
        total += F.total[k];
    }
    const size_t lds = std::max({sweep_lds_bytes(256), bt.rowLds, VISC ? sizeof(ViscLds<double, DIAG>) : 0});
    const dim3 g(grid_for(total)), b(256);
    if (bt.weights == CNS_WENO_Z) hipLaunchKernelGGL((k_small<VISC, DIAG, CNS_WENO_Z>), g, b, lds, bt.stream, L, F);
    else if (bt.weights == CNS_WENO_M) hipLaunchKernelGGL((k_small<VISC, DIAG, CNS_WENO_M>), g, b, lds, bt.stream, L, F);
    else hipLaunchKernelGGL((k_small<VISC, DIAG, CNS_WENO_JS>), g, b, lds, bt.stream, L, F);
}

template <int MODE>
static void stage_sum(const Batch &bt, const Launch &L) {
    const dim3 g(grid_for(L.total)), b(kPointThreads);
    if (bt.any_visc) hipLaunchKernelGGL((k_stage_sum<MODE, true>), g, b, 0, bt.stream, L);
    else hipLaunchKernelGGL((k_stage_sum<MODE, false>), g, b, 0, bt.stream, L);
}

// L.stage 0: the right-hand side; diag_prev as in first_visc
static void small_stage_run(const Batch &bt, Launch L, double *diag = nullptr, long long stride = 0, int diag_prev = -1) {
    L = with_family(bt, L, F_POINT);
    if (bt.any_visc && diag_prev >= 0) {
        Launch D = L;
        D.diag = diag;
        D.diag_box_stride = stride;
        D.step = diag_prev;
        D.diag_fused = 1;
        small_sweeps<true, true>(bt, D);
        D = with_family(bt, D, F_BOX);
        hipLaunchKernelGGL(k_diag_final, dim3(grid_for(D.total)), dim3(kDiagThreads), 0, bt.stream, D);
    } else if (bt.any_visc) {
        small_sweeps<true, false>(bt, L);
    } else {
        small_sweeps<false, false>(bt, L);
    }
    if (L.stage == 0) stage_sum<MODE_ACCUM>(bt, L);
    else if (L.stage == 1) stage_sum<MODE_RK1>(bt, L);
    else if (L.scheme == CNS_RK4 && L.stage == 4) stage_sum<MODE_RK3>(bt, L);
    else stage_sum<MODE_RK2>(bt, L);
}

template <typename T>
static void rhs_t(const Batch &bt, const void *u_ov, void *out_ov) {
    Launch L = make_launch(bt, F_POINT);
    L.in = BUF_U;
    L.u_ov = u_ov;
    L.out_ov = out_ov;
    if (small_stage(bt)) return small_stage_run(bt, L);
    if (bt.any_visc) visc_fields<T>(bt, L);
    sweep_x<T>(bt, L, bt.any_visc);
    {
        ProfScope ps(bt.prof, K_SWEEP_Y, bt.stream);
        sweep<T, MODE_ACCUM>(bt, L, 1, bt.any_visc);
    }
    ProfScope ps(bt.prof, K_SWEEP_Z, bt.stream);
    sweep<T, MODE_ACCUM>(bt, L, 2, bt.any_visc);
}

void launch_rhs(const Batch &bt, const void *u_ov, void *out_ov) {
    if (bt.prec == CNS_FP64) rhs_t<double>(bt, u_ov, out_ov);
    else rhs_t<float>(bt, u_ov, out_ov);
}

template <typename T>
static void rhs_dir_t(const Batch &bt, const void *u_ov, int dir, void *out_ov) {
    Launch L = make_launch(bt, F_POINT);
    L.in = BUF_U;
    L.u_ov = u_ov;
    L.out_ov = out_ov;
    if (dir == 0) sweep_x<T>(bt, L, false);
    else sweep<T, MODE_WRITE>(bt, L, dir, false);
}

void launch_rhs_dir(const Batch &bt, const void *u_ov, int dir, void *out_ov) {
    if (bt.prec == CNS_FP64) rhs_dir_t<double>(bt, u_ov, dir, out_ov);
    else rhs_dir_t<float>(bt, u_ov, dir, out_ov);
}

template <typename T>
static void viscous_t(const Batch &bt, const void *u_ov, void *out_ov) {
    Launch L = make_launch(bt, F_POINT);
    L.in = BUF_U;
    L.u_ov = u_ov;
    if constexpr (kMixed<T>) {
        L.out_ov = out_ov;
        mixed::viscous(bt, L);
    } else {
        // rows 1-4 of the output; the density row has no viscous term
        const BoxDesc &b = *bt.box0;
        L.v_ov = (T *)out_ov + b.n3;
        launch_fill(bt.prec, b.n3, out_ov, bt.stream);
        // alone on the chip, with no sweeps beside it: fewer planes per block than in a stage
        // while that leaves CUs without one (8 x 128 x 128: 42 us with 16 planes, 26 with 8;
        // 112^3: 58 us with 16, 66 with 8)
        L = with_family(bt, L, F_VISC);
        L.vsz_ov = b.vsz;
        while (L.vsz_ov > 2 && plane_tiles(b.nx, b.ny, b.nz, L.vsz_ov) < 256) L.vsz_ov /= 2;
        L.total = plane_tiles(b.nx, b.ny, b.nz, L.vsz_ov);
        hipLaunchKernelGGL((k_visc<T, false>), dim3(grid_for(L.total)), dim3(ViscTile<T>::kThreads), 0, bt.stream, L);
    }
}

void launch_viscous(const Batch &bt, const void *u_ov, void *out_ov) {
    if (bt.prec == CNS_FP64) viscous_t<double>(bt, u_ov, out_ov);
    else viscous_t<float>(bt, u_ov, out_ov);
}

template <typename T>
static void diag_t(const Batch &bt, const void *u_ov, double *diag, long long stride, int step) {
    ProfScope ps(bt.prof, K_DIAG, bt.stream);
    Launch L = make_launch(bt, F_DIAG);
    L.u_ov = u_ov;
    L.diag = diag;
    L.diag_box_stride = stride;
    L.step = step;
    const dim3 g(grid_of(bt, F_DIAG, L.total)), b(kDiagThreads);
    const bool three = sizeof(T) == 8 && g.x <= 3 * 256;  // three on each of 256 CUs
    if constexpr (sizeof(T) == 8)
        if (three) hipLaunchKernelGGL((k_diag_partial<T, 3>), g, b, 0, bt.stream, L);
    if (!three) hipLaunchKernelGGL((k_diag_partial<T, 4>), g, b, 0, bt.stream, L);
    const Launch F = with_family(bt, L, F_BOX);
    hipLaunchKernelGGL(k_diag_final, dim3(grid_for(F.total)), dim3(kDiagThreads), 0, bt.stream, F);
}

void launch_max_wave_speed(const Batch &bt, const void *u_ov, double *out) {
    Launch L = make_launch(bt, F_DIAG);
    L.u_ov = u_ov;
    if (bt.prec == CNS_FP64)
        hipLaunchKernelGGL(k_speed_partial<double>, dim3(grid_for(L.total)), dim3(kDiagThreads), 0, bt.stream, L);
    else
        hipLaunchKernelGGL(k_speed_partial<float>, dim3(grid_for(L.total)), dim3(kDiagThreads), 0, bt.stream, L);
    const Launch F = with_family(bt, L, F_BOX);
    hipLaunchKernelGGL(k_speed_final, dim3(grid_for(F.total)), dim3(kDiagThreads), 0, bt.stream, F, out);
}

void launch_stream_copy(const void *src, void *dst, size_t bytes, hipStream_t s) {
    const size_t n16 = bytes / 16;
    // 8 blocks of 256 threads per CU on the 256 CUs
    const unsigned g = (unsigned)std::min<size_t>((n16 + 255) / 256, 2048);
    if (n16) hipLaunchKernelGGL(k_stream_copy, dim3(g), dim3(256), 0, s, (const v2d *)src, (v2d *)dst, n16);
}

void launch_set_params(GraphParams *gp, const void *u, double *diag, double dt, hipStream_t s) {
    hipLaunchKernelGGL(k_set_params, dim3(1), dim3(64), 0, s, gp, u, diag, dt);
}

void launch_diag(const Batch &bt, const void *u_ov, double *diag, long long stride, int step) {
    if (bt.prec == CNS_FP64) diag_t<double>(bt, u_ov, diag, stride, step);
    else diag_t<float>(bt, u_ov, diag, stride, step);
}

// the device table of one box, written from a kernel argument (no host-to-device copy)
__global__ void k_write_table(OneBoxTable t, OneBoxTable *dst) {
    if (threadIdx.x == 0 && blockIdx.x == 0) *dst = t;
}

size_t static_diag_bytes() { return align_up256(sizeof(OneBoxTable)) + (size_t)kDiagBlocksMax * CNS_NDIAG * sizeof(double); }

void launch_diag_static(char *scratch_dev, const BoxDesc &b, int prec, const void *u, double *out, hipStream_t s) {
    OneBoxTable t{};
    t.b = b;
    t.b.part = (double *)(scratch_dev + align_up256(sizeof(OneBoxTable)));
    for (int f = 0; f < F_N; ++f) {
        t.off[f][0] = 0;
        t.off[f][1] = family_blocks(t.b, f, 256);
    }
    OneBoxTable *dt = (OneBoxTable *)scratch_dev;
    hipLaunchKernelGGL(k_write_table, dim3(1), dim3(64), 0, s, t, dt);
    Batch bt;
    bt.nbox = 1;
    bt.prec = prec;
    bt.d_boxes = &dt->b;
    for (int f = 0; f < F_N; ++f) {
        bt.d_off[f] = dt->off[f];
        bt.total[f] = t.off[f][1];
    }
    bt.stream = s;
    launch_diag(bt, u, out, 0, 0);
}



// The first stage's viscous-flux launch of a step, forming the diagnostics of the state
// it reads (record diag_prev) when diag_prev >= 0 (FP64, viscous batches), then their
// per-box reduction.
template <typename T>
static void first_visc(const Batch &bt, Launch L, double *diag, long long stride, int diag_prev) {
    if constexpr (std::is_same<T, double>::value) {
        if (diag_prev >= 0) {
            L.diag = diag;
            L.diag_box_stride = stride;
            L.step = diag_prev;
            L.diag_fused = 1;
            visc_fields<T, true>(bt, L);
            const Launch F = with_family(bt, L, F_BOX);
            hipLaunchKernelGGL(k_diag_final, dim3(grid_for(F.total)), dim3(kDiagThreads), 0, bt.stream, F);
            return;
        }
    }
    visc_fields<T>(bt, L);
}

template <typename T>
static void rk4_step_t(const Batch &bt, const void *u_ov, double dt_ov, double *diag, long long stride, int step,
                       void *const *stage_states, int diag_prev, bool diag_own) {
    // stage s reads U_s and writes U_{s+1}: U_1 = u, U_2 -> A, U_3 -> B, U_4 -> A, u^{n+1} -> u;
    // with stage_states, A is U2's buffer for stages 1-2 and U4's for stages 3-4, B is U3's
    const int in_of[4] = {BUF_U, BUF_A, BUF_B, BUF_A};
    const int out_of[4] = {BUF_A, BUF_B, BUF_A, BUF_U};
    for (int s = 0; s < 4; ++s) {
        Launch L = make_launch(bt, F_POINT);
        L.in = in_of[s];
        L.out = out_of[s];
        L.stage = s + 1;
        L.u_ov = u_ov;
        if (stage_states) {
            L.a_ov = stage_states[s < 2 ? 0 : 2];
            L.b_ov = stage_states[1];
        }
        L.dt_ov = dt_ov;
        if (small_stage(bt)) {
            small_stage_run(bt, L, diag, stride, s == 0 ? diag_prev : -1);
            continue;
        }
        if (bt.any_visc) {
            if (s == 0) first_visc<T>(bt, L, diag, stride, diag_prev);
            else visc_fields<T>(bt, L);
        }
        sweep_x<T>(bt, L, bt.any_visc);
        {
            ProfScope ps(bt.prof, K_SWEEP_Y, bt.stream);
            sweep<T, MODE_ACCUM>(bt, L, 1, bt.any_visc);
        }
        ProfScope ps(bt.prof, K_SWEEP_Z, bt.stream);
        sweep_rk<T>(bt, L);
    }
    if (diag && diag_own) diag_t<T>(bt, u_ov, diag, stride, step);
}

void launch_rk4_step(const Batch &bt, const void *u_ov, double dt_ov, double *diag, long long stride, int step,
                     void *const *stage_states, int diag_prev, bool diag_own) {
    if (bt.prec == CNS_FP64) rk4_step_t<double>(bt, u_ov, dt_ov, diag, stride, step, stage_states, diag_prev, diag_own);
    else rk4_step_t<float>(bt, u_ov, dt_ov, diag, stride, step, stage_states, diag_prev, diag_own);
}

template <typename T>
static void tvdrk3_step_t(const Batch &bt, const void *u_ov, double dt_ov, double *diag, long long stride,
                          int step, void *const *stage_states, int diag_prev, bool diag_own) {
    // stage s reads U_s and writes U_{s+1}: U_1 = u, U_2 -> A, U_3 -> B, u^{n+1} -> u;
    // with stage_states, A is stage_states[0] and B stage_states[1]
    const int in_of[3] = {BUF_U, BUF_A, BUF_B};
    const int out_of[3] = {BUF_A, BUF_B, BUF_U};
    for (int s = 0; s < 3; ++s) {
        Launch L = make_launch(bt, F_POINT);
        L.in = in_of[s];
        L.out = out_of[s];
        L.stage = s + 1;
        L.scheme = CNS_TVDRK3;
        L.u_ov = u_ov;
        L.dt_ov = dt_ov;
        if (stage_states) {
            L.a_ov = stage_states[0];
            L.b_ov = stage_states[1];
        }
        if (small_stage(bt)) {
            small_stage_run(bt, L, diag, stride, s == 0 ? diag_prev : -1);
            continue;
        }
        if (bt.any_visc) {
            if (s == 0) first_visc<T>(bt, L, diag, stride, diag_prev);
            else visc_fields<T>(bt, L);
        }
        sweep_x<T>(bt, L, bt.any_visc);
        {
            ProfScope ps(bt.prof, K_SWEEP_Y, bt.stream);
            sweep<T, MODE_ACCUM>(bt, L, 1, bt.any_visc);
        }
        ProfScope ps(bt.prof, K_SWEEP_Z, bt.stream);
        sweep_rk<T>(bt, L);
    }
    if (diag && diag_own) diag_t<T>(bt, u_ov, diag, stride, step);
}

void launch_step(const Batch &bt, int scheme, const void *u_ov, double dt_ov, double *diag, long long stride,
                 int step, void *const *stage_states, int diag_prev, bool diag_own) {
    if (scheme == CNS_RK4)
        return launch_rk4_step(bt, u_ov, dt_ov, diag, stride, step, stage_states, diag_prev, diag_own);
    if (bt.prec == CNS_FP64)
        tvdrk3_step_t<double>(bt, u_ov, dt_ov, diag, stride, step, stage_states, diag_prev, diag_own);
    else tvdrk3_step_t<float>(bt, u_ov, dt_ov, diag, stride, step, stage_states, diag_prev, diag_own);
}

float time_sweeps_yz(const Batch &bt, int reps) {
    hipEvent_t a, b;
    (void)hipEventCreate(&a);
    (void)hipEventCreate(&b);
    Launch L = make_launch(bt, F_POINT);
    L.in = BUF_U;
    (void)hipEventRecord(a, bt.stream);
    for (int r = 0; r < reps; ++r) {
        if (bt.prec == CNS_FP64) {
            sweep<double, MODE_WRITE>(bt, L, 1, bt.any_visc);
            sweep<double, MODE_WRITE>(bt, L, 2, bt.any_visc);
        } else {
            sweep<float, MODE_WRITE>(bt, L, 1, bt.any_visc);
            sweep<float, MODE_WRITE>(bt, L, 2, bt.any_visc);
        }
    }
    (void)hipEventRecord(b, bt.stream);
    (void)hipEventSynchronize(b);
    float ms = 0.f;
    (void)hipEventElapsedTime(&ms, a, b);
    (void)hipEventDestroy(a);
    (void)hipEventDestroy(b);
    return ms / (float)(reps > 0 ? reps : 1);
}

float time_rhs_kernels(const Batch &bt, int reps) {
    hipEvent_t a, b;
    (void)hipEventCreate(&a);
    (void)hipEventCreate(&b);
    (void)hipEventRecord(a, bt.stream);
    for (int r = 0; r < reps; ++r) launch_rhs(bt, nullptr, nullptr);
    (void)hipEventRecord(b, bt.stream);
    (void)hipEventSynchronize(b);
    float ms = 0.f;
    (void)hipEventElapsedTime(&ms, a, b);
    (void)hipEventDestroy(a);
    (void)hipEventDestroy(b);
    return ms / (float)(reps > 0 ? reps : 1);
}

static long long cu_count() {
    int dev = 0, cus = 0;
    if (hipGetDevice(&dev) != hipSuccess || hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) !=
                                                 hipSuccess)
        return 256;
    return cus;
}

long long resident_sweep_blocks(const Batch &bt) {
    int n = 0;
    if (bt.prec != CNS_FP64) n = mixed::resident_sweep_blocks(bt.block);
    else if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, k_sweep<double, 2, MODE_RK2, false, CNS_WENO_JS>, bt.block,
                                                          sweep_lds_bytes(bt.block)) != hipSuccess)
        n = 0;
    return (n > 0 ? n : 1) * cu_count();
}

long long resident_tile_blocks(const Batch &bt) {
    int n = 0;
    if (bt.prec != CNS_FP64) n = mixed::resident_tile_blocks();
    else if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, k_visc<double, false>, ViscTile<double>::kThreads, 0) !=
             hipSuccess)
        n = 0;
    return (n > 0 ? n : 1) * cu_count();
}

void prof_flush(Prof *p) {
    if (!p || !p->on || p->n == 0) return;
    (void)hipEventSynchronize(p->ev[2 * p->n - 1]);
    for (int i = 0; i < p->n; ++i) {
        float ms = 0.f;
        if (hipEventElapsedTime(&ms, p->ev[2 * i], p->ev[2 * i + 1]) == hipSuccess) {
            p->ms[p->kind[i]] += ms;
            p->count[p->kind[i]] += 1;
        }
    }
    p->n = 0;
}

}  // namespace cns
