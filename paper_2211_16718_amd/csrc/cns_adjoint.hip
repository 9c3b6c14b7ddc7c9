// cns_adjoint.hip -- reverse-mode kernels of the RHS (vector-Jacobian products) and the
// small kernels of the checkpointed reverse RK4, FP64, single box.
//
// (dR/du)^T rbar of the semi-discrete operator R(u) = -sum_d (H_{j+1/2} - H_{j-1/2})/dx_d
// + sum_d D_d G^v_d is assembled as
//   convective part, per direction d:  Hbar_{j+1/2} = (rbar_{j+1} - rbar_j)/dx_d;
//     k_adj_cells, k_adj_march: a lane per cell, or a thread marching from cell to cell,
//     transposes the cell's reconstructions and a face's dissipation and adds the
//     point-flux and state adjoints of the cells, which are then finished and written;
//   viscous part: the adjoint of a central difference is minus the same central
//     difference, so Gbar_d = -D_d rbar; k_adj_visc maps it through the viscous
//     fluxes to the adjoints of the velocity/temperature gradients and of the
//     point velocities, applies -D once more and the primitive map, in one pass.
// Every sum is formed in a fixed order (deterministic: the LDS additions into a cell
// come from one wave, whose LDS operations take effect in program order).
#include <hip/hip_runtime.h>

#include "cns_adjoint.h"
#include "cns_batch.h"
#include "cns_device_adj.h"
#include "cns_internal.h"

namespace cns {

__device__ __forceinline__ int wrapj(int j, int n) { return j < 0 ? j + n : (j >= n ? j - n : j); }
// any number of periods (the halo of a 64-wide tile over a shorter line)
__device__ __forceinline__ int wrapn(int j, int n) {
    const int r = j % n;
    return r < 0 ? r + n : r;
}

struct AdjGeom {
    int nx, ny, nz;
    size_t n3;
    double ih[3];
    double gamma, prandtl, mu, eps, delta;
};

static AdjGeom adj_geom(const BoxDesc &b) {
    AdjGeom g;
    g.nx = b.nx;
    g.ny = b.ny;
    g.nz = b.nz;
    g.n3 = b.n3;
    for (int d = 0; d < 3; ++d) g.ih[d] = b.inv_h[d];
    g.gamma = b.gamma;
    g.prandtl = b.prandtl;
    g.mu = b.mu;
    g.eps = b.eps;
    g.delta = b.delta;
    return g;
}

// ---------------------------------------------------------------------------
// Convective adjoint along DIR = y or z by cells: ubar += the terms of every cell's
// reconstructions and of every face's dissipation.
//
// A thread marches over a segment s0 .. s1-1 of one periodic line.  In step j it transposes
// the nine reconstructions of cell j (the state and the fluxes 1-4; the mass flux is the
// momentum along the line, so its adjoint joins that component's), for which it has formed
// dub = M^T Db of the right face from the states j, j+1, and the left face's a step before;
// the values then give the jump at the left face, whose dissipation is transposed for the
// states j-1, j.  A reconstruction's terms go to cells j-2 .. j+2: the sums of the four
// cells not yet complete stay in registers and move up one place as they are added to;
// cell j-2 is complete, and leaves as J^T F + U (J the flux Jacobian: once per cell).
// Nothing is shared between threads, so the march has no barrier: LDS holds each thread's
// own window of five cells (state, normal velocity, pressure) and dub.
//
// Segments meet without redundant cells.  A thread adds to ubar cells s0-2 .. s1-3 during
// its march, and after a barrier (the segments of a line are in one block) the sums of
// cells s1-2 .. s1+1 that it still holds; a segment is at least four cells long, so in
// either phase no two threads touch the same cell.  The face between two segments is the
// left one's: it forms the right-biased values of cell s1 again.
//
// Bound by FP64 issue: 1440 instructions a step at 78 % of the issue rate, two waves per SIMD
// (the sums and face values take all 256 registers).  128^3: 167 us, 215 with a thread per
// interface, six-point stencils and the sums in LDS; 130 x 90 x 66: 86 against 117.
// ---------------------------------------------------------------------------
constexpr int kAmThreads = 256;
constexpr int kAmCells = 5, kAmComp = 7;  // cells of the window, scalars of a cell

template <int DIR, int WW>
__global__ __launch_bounds__(kAmThreads, 2) void k_adj_march(AdjGeom g, const double *u_,
                                                             const double *rbar_, double *ubar_, int Lb,
                                                             int nseg) {
    __shared__ double win[(kAmCells * kAmComp + 5) * kAmThreads];  // 80 KiB: two blocks on a CU
    constexpr int NT = kAmThreads;
    const auto u = (gptr<const double>)u_, rbar = (gptr<const double>)rbar_;
    const auto ubar = (gptr<double>)ubar_;
    const int t = threadIdx.x, seg = t / Lb;
    const size_t n3 = g.n3, nlines = DIR == 1 ? (size_t)g.nx * g.nz : (size_t)g.nx * g.ny;
    const size_t line = (size_t)blockIdx.x * Lb + (t - seg * Lb);
    const int n = DIR == 1 ? g.ny : g.nz;
    // byte offsets within a component
    const uint32_t stride = (uint32_t)(8 * (DIR == 1 ? (size_t)g.nx : (size_t)g.nx * g.ny));
    const uint32_t base = (uint32_t)(8 * (DIR == 1 ? line / g.nx * ((size_t)g.nx * g.ny) + line % g.nx : line));
    const bool ok = seg < nseg && line < nlines;
    const int s0 = (int)((long long)seg * n / nseg), s1 = (int)((long long)(seg + 1) * n / nseg);
    const int len = ok ? s1 - s0 : 0, kmax = (n + nseg - 1) / nseg;
    const double ih12 = g.ih[DIR] * (1.0 / 12.0), gm1 = g.gamma - 1.0, eps4 = 4.0 * g.eps;
    double *const dubL = win + kAmCells * kAmComp * NT + t;  // dub of the left face
    auto at = [&](int slot, int v) -> double & { return win[(slot * kAmComp + v) * NT + t]; };
    auto cell = [&](int j) { return base + (uint32_t)wrapj(j, n) * stride; };
    auto load5 = [&](gptr<const double> p, uint32_t c, double w[5]) {
#pragma unroll
        for (int v = 0; v < 5; ++v) w[v] = *elem(p, n3, v, c);
    };
    auto keep = [&](int slot, const double w[5]) {
        const double inv = rcp(w[0]), vx = w[1] * inv, vy = w[2] * inv, vz = w[3] * inv;
#pragma unroll
        for (int v = 0; v < 5; ++v) at(slot, v) = w[v];
        at(slot, 5) = DIR == 1 ? vy : vz;
        at(slot, 6) = gm1 * (w[4] - 0.5 * (w[1] * vx + w[2] * vy + w[3] * vz));
    };
    auto states = [&](int sa, int sb, double a[5], double b[5]) {
#pragma unroll
        for (int v = 0; v < 5; ++v) a[v] = at(sa, v), b[v] = at(sb, v);
    };
    // Everything per face is held for six times the reconstructed values: H = Hbar / 12, dub =
    // M^T Db / 6 = -M^T H, the jumps 6 du with H in place of Hbar / 2.
    // -M^T H of the face between the cells at sa and sb
    auto jump_adjoint = [&](int sa, int sb, const double H[5], double dub[5]) {
        double a[5], b[5], Db[5];
        states(sa, sb, a, b);
#pragma unroll
        for (int v = 0; v < 5; ++v) Db[v] = -H[v], dub[v] = 0.0;
        const RoeFace R = roe_face<DIR>(a, at(sa, 6), b, at(sb, 6), gm1, g.delta);
        roe_jump_vjp<DIR>(R, gm1, Db, dub);
    };
    double AU[4][5], AF[4][4];  // sums of cells j-2 .. j+1 before step j
    double UL[5], Hl[5];        // six times the left-biased values, and H, of the left face
    auto state_adjoint = [&](int sa, int sb, double h, const double du6[5], double ab[5], double bb[5]) {
        double a[5], b[5], Db[5];
        states(sa, sb, a, b);
#pragma unroll
        for (int v = 0; v < 5; ++v) Db[v] = h * Hl[v];
        const RoeFace R = roe_face<DIR>(a, at(sa, 6), b, at(sb, 6), gm1, g.delta);
        double vbar[3], Hbar;
        roe_mean_vjp<DIR>(R, gm1, g.delta, du6, Db, vbar, Hbar);
        pin(vbar[0]), pin(vbar[1]), pin(vbar[2]), pin(Hbar);
        adj_stage_fence();
        states(sa, sb, a, b);
        roe_cells_vjp(R, a, at(sa, 6), b, at(sb, 6), gm1, vbar, Hbar, ab, bb);
    };
    // ubar at q += J^T f + us, J of the cell at slot
    auto finish = [&](int slot, const double us[5], const double f[4], const double old[5], uint32_t q) {
        double w[5], fb[5] = {0.0, f[0], f[1], f[2], f[3]}, out[5];
#pragma unroll
        for (int v = 0; v < 5; ++v) w[v] = at(slot, v), out[v] = us[v];
        euler_flux_vjp<DIR>(w, gm1, fb, out);
#pragma unroll
        for (int v = 0; v < 5; ++v) *elem(ubar, n3, v, q) = old[v] + out[v];
    };
    double rb[5], rn[5];  // rbar of cells j and j+1
    if (ok) {
        double w[kAmCells][5], rm[5];
#pragma unroll
        for (int m = 0; m < kAmCells; ++m) load5(u, cell(s0 - 2 + m), w[m]);
        load5(rbar, cell(s0 - 1), rm);
        load5(rbar, cell(s0), rb);
        load5(rbar, cell(s0 + 1), rn);
#pragma unroll
        for (int m = 0; m < kAmCells; ++m) keep(m, w[m]);
        double dub[5];
#pragma unroll
        for (int v = 0; v < 5; ++v) Hl[v] = (rb[v] - rm[v]) * ih12, UL[v] = 0.0;
        jump_adjoint(1, 2, Hl, dub);
#pragma unroll
        for (int v = 0; v < 5; ++v) dubL[v * NT] = dub[v];
#pragma unroll
        for (int m = 0; m < 4; ++m) {
#pragma unroll
            for (int v = 0; v < 5; ++v) AU[m][v] = 0.0;
#pragma unroll
            for (int v = 0; v < 4; ++v) AF[m][v] = 0.0;
        }
    }
    int o0 = 0, o1 = 1, o2 = 2, o3 = 3, o4 = 4;  // slots of cells j-2 .. j+2
    for (int k = 0; k < kmax; ++k) {
        if (k < len) {
            const int j = s0 + k;
            double Hr[5], dub[5], du[5], dU[5], dF[4], old[5], un[5];  // un: state of cell j+3
#pragma unroll
            for (int v = 0; v < 5; ++v) Hr[v] = (rn[v] - rb[v]) * ih12, rb[v] = rn[v], pin(Hr[v]);
            const int o[5] = {o0, o1, o2, o3, o4};
            double x[5], xn[5], xb[5], L6, R6;
            // the fluxes; each component's loads from LDS are issued one component ahead
            {
                double vn[5], p[5];
#pragma unroll
                for (int m = 0; m < 5; ++m) vn[m] = at(o[m], 5), xn[m] = at(o[m], 1);
#pragma unroll
                for (int v = 1; v < 5; ++v) {
#pragma unroll
                    for (int m = 0; m < 5; ++m) {
                        x[m] = xn[m] * vn[m];
                        if (v == 1 + DIR) x[m] += at(o[m], 6);
                        if (v == 4) x[m] += p[m] * vn[m];
                        if (v < 4) xn[m] = at(o[m], v + 1);
                        if (v == 3) p[m] = at(o[m], 6);
                    }
                    adj_stage_fence();
                    weno5_cell_vjp<WW>(x, eps4, Hr[v], Hl[v], xb, L6, R6);
                    dF[v - 1] = AF[0][v - 1] + xb[0];
#pragma unroll
                    for (int m = 0; m < 3; ++m) AF[m][v - 1] = AF[m + 1][v - 1] + xb[m + 1];
                    AF[3][v - 1] = xb[4];
                    pin(dF[v - 1]);
#pragma unroll
                    for (int m = 0; m < 4; ++m) pin(AF[m][v - 1]);
                    adj_stage_fence();
                }
            }
            jump_adjoint(o2, o3, Hr, dub);
#pragma unroll
            for (int v = 0; v < 5; ++v) pin(dub[v]);
            adj_stage_fence();
            // the states, with the mass flux's terms in the momentum along the line
            double dl = dubL[0];
#pragma unroll
            for (int m = 0; m < 5; ++m) xn[m] = at(o[m], 0);
#pragma unroll
            for (int v = 0; v < 5; ++v) {
#pragma unroll
                for (int m = 0; m < 5; ++m) x[m] = xn[m];
                double Lb = -dub[v], Rb = dl;
                dubL[v * NT] = dub[v];
                if (v == 1 + DIR) Lb += Hr[0], Rb += Hl[0];
                if (v < 4) {
#pragma unroll
                    for (int m = 0; m < 5; ++m) xn[m] = at(o[m], v + 1);
                    dl = dubL[(v + 1) * NT];
                }
                if (v == 1) load5(u, cell(j + 3), un);
                if (v == 2) load5(ubar, cell(j - 2), old);
                if (v == 4) load5(rbar, cell(j + 2), rn);
                adj_stage_fence();
                weno5_cell_vjp<WW>(x, eps4, Lb, Rb, xb, L6, R6);
                du[v] = R6 - UL[v];
                UL[v] = L6;
                dU[v] = AU[0][v] + xb[0];
#pragma unroll
                for (int m = 0; m < 3; ++m) AU[m][v] = AU[m + 1][v] + xb[m + 1];
                AU[3][v] = xb[4];
                pin(du[v]), pin(UL[v]), pin(dU[v]);
#pragma unroll
                for (int m = 0; m < 4; ++m) pin(AU[m][v]);
                adj_stage_fence();
            }
            finish(o0, dU, dF, old, cell(j - 2));
            keep(o0, un);
            adj_stage_fence();
            state_adjoint(o1, o2, k > 0 ? -1.0 : 0.0, du, AU[0], AU[1]);
#pragma unroll
            for (int v = 0; v < 5; ++v) pin(AU[0][v]), pin(AU[1][v]);
#pragma unroll
            for (int v = 0; v < 5; ++v) Hl[v] = Hr[v];
        }
        const int f = o0;
        o0 = o1, o1 = o2, o2 = o3, o3 = o4, o4 = f;
    }
    int e0 = len % kAmCells;  // slot of cell s1-2
    auto slot_of = [&](int m) { return e0 + m >= kAmCells ? e0 + m - kAmCells : e0 + m; };
    if (ok) {
        double du[5];
#pragma unroll
        for (int v = 0; v < 5; ++v) {
            // (the values of the product itself: its range is wider than the forward form's)
            double x[5], xb[5], L6, R6;
#pragma unroll
            for (int m = 0; m < 5; ++m) x[m] = at(slot_of(m), v);
            weno5_cell_vjp<WW>(x, eps4, 0.0, 0.0, xb, L6, R6);
            du[v] = R6 - UL[v];
        }
        state_adjoint(slot_of(1), slot_of(2), -1.0, du, AU[1], AU[2]);
    }
    __syncthreads();
    if (!ok) return;
#pragma unroll
    for (int m = 0; m < 4; ++m) {
        const uint32_t q = cell(s1 - 2 + m);
        double old[5];
        load5(ubar, q, old);
        finish(slot_of(m), AU[m], AF[m], old, q);
    }
}

// ---------------------------------------------------------------------------
// Convective adjoint with a lane per cell, along x and in small boxes along y and z: ubar = (x)
// or += the same terms.  A wave takes chunks of 16 cells of four segments of lines (x: loads of
// whole 128-byte pieces), with the segments, their two phases and their faces as in the march.  What a thread of the march
// keeps in registers is in LDS, private to the wave, so that no barrier orders it: the sums of
// the chunk's cells and two on either side (LDS additions: one instruction adds to sixteen
// different cells of a segment, so their order is fixed), dub and the left-biased values at a
// slot per face, and the states, pressures and rbar of the chunk, whose next cells are
// loaded a chunk ahead.
//
// SPARE: where a segment's last chunk leaves lanes idle, the one past its end forms the last
// face with the chunk, as the lane of a cell whose reconstructions carry nothing; otherwise
// one lane forms it after the chunks.  In small boxes, whose launches last as long as one
// segment, that is a quarter of the time (16^3, three directions 39.8 -> 28.2 us); large ones do
// not wait for it and would pay the products by zero (128^3, WENO-Z: 712 -> 730 us).
//
// Bound by FP64 issue (75 % of the rate) and LDS (47 % busy), two waves per SIMD.  128^3 along
// x: 181 us against 215 with a lane per interface; 130 x 90 x 66: 92 against 117.
// ---------------------------------------------------------------------------
constexpr int kAcTA = 16, kAcLW = 4;            // cells of a chunk, segments of a wave
constexpr int kAcNC = kAcTA + 5;                // staged cells I-2 .. I+TA+2
constexpr int kAcKA = kAcTA + 4;                // summed cells I-2 .. I+TA+1
constexpr int kAcSeg = 4 * kAcLW;               // segments of a block
constexpr int kAcWave = (12 * kAcNC + 9 * kAcKA + 10 * (kAcTA + 1)) * kAcLW;

template <int DIR, int WW, bool SPARE>
__global__ __launch_bounds__(256, 2) void k_adj_cells(AdjGeom g, const double *u_, const double *rbar_, double *ubar_,
                                                      int nseg) {
    constexpr int TA = kAcTA, LW = kAcLW, NC = kAcNC, KA = kAcKA;
    __shared__ double lds[4 * kAcWave];
    const auto u = (gptr<const double>)u_, rbar = (gptr<const double>)rbar_;
    const auto ubar = (gptr<double>)ubar_;
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6, ta = lane / LW, tl = lane % LW;
    const int lb = kAcSeg / nseg, vs = wv * LW + tl, seg = vs / lb;
    const size_t n3 = g.n3, line = (size_t)blockIdx.x * lb + vs % lb;
    const size_t nlines = DIR == 0 ? (size_t)g.ny * g.nz : (DIR == 1 ? (size_t)g.nx * g.nz : (size_t)g.nx * g.ny);
    const int n = DIR == 0 ? g.nx : (DIR == 1 ? g.ny : g.nz);
    const bool ok = line < nlines;
    // byte offsets within a component
    const uint32_t stride = (uint32_t)(8 * (DIR == 0 ? (size_t)1 : (DIR == 1 ? (size_t)g.nx : (size_t)g.nx * g.ny)));
    const uint32_t base = (uint32_t)(8 * (DIR == 0 ? line * n
                                                   : (DIR == 1 ? line / g.nx * ((size_t)g.nx * g.ny) + line % g.nx : line)));
    const int s0 = (int)((long long)seg * n / nseg), s1 = ok ? (int)((long long)(seg + 1) * n / nseg) : s0;
    const double ih12 = g.ih[DIR] * (1.0 / 12.0), gm1 = g.gamma - 1.0, eps4 = 4.0 * g.eps;
    double *const sw = lds + wv * kAcWave + tl;
    // staged scalar v of staged cell c (0-4 the state, 5 normal velocity, 6 pressure, 7-11 rbar),
    // sum v of summed cell c (0-4 state, 5-8 fluxes 1-4), dub and left-biased value v of face slot c
    auto S = [&](int v, int c) -> double & { return sw[(v * NC + c) * LW]; };
    auto A = [&](int v, int c) -> double & { return sw[(12 * NC + v * KA + c) * LW]; };
    auto D = [&](int v, int c) -> double & { return sw[(12 * NC + 9 * KA + v * (TA + 1) + c) * LW]; };
    auto UL = [&](int v, int c) -> double & { return sw[(12 * NC + 9 * KA + (5 + v) * (TA + 1) + c) * LW]; };
    auto cell = [&](int j) { return base + (uint32_t)wrapn(j, n) * stride; };
    auto load5 = [&](gptr<const double> p, uint32_t c, double w[5]) {
#pragma unroll
        for (int v = 0; v < 5; ++v) w[v] = *elem(p, n3, v, c);
    };
    auto keep = [&](int c, const double w[5], const double r[5]) {
        const double inv = rcp(w[0]), vx = w[1] * inv, vy = w[2] * inv, vz = w[3] * inv;
#pragma unroll
        for (int v = 0; v < 5; ++v) S(v, c) = w[v], S(7 + v, c) = r[v];
        S(5, c) = DIR == 0 ? vx : (DIR == 1 ? vy : vz);
        S(6, c) = gm1 * (w[4] - 0.5 * (w[1] * vx + w[2] * vy + w[3] * vz));
    };
    auto states = [&](int c, double a[5], double b[5]) {
#pragma unroll
        for (int v = 0; v < 5; ++v) a[v] = S(v, c), b[v] = S(v, c + 1);
    };
    auto jump_adjoint = [&](int c, const double H[5], double dub[5]) {  // as in the march; the face of cells c, c + 1
        double a[5], b[5], Db[5];
        states(c, a, b);
#pragma unroll
        for (int v = 0; v < 5; ++v) Db[v] = -H[v], dub[v] = 0.0;
        const RoeFace R = roe_face<DIR>(a, S(6, c), b, S(6, c + 1), gm1, g.delta);
        roe_jump_vjp<DIR>(R, gm1, Db, dub);
    };
    auto state_adjoint = [&](int c, const double Db[5], const double du6[5], double ab[5], double bb[5]) {
        double a[5], b[5], vbar[3], Hbar;
        states(c, a, b);
        const RoeFace R = roe_face<DIR>(a, S(6, c), b, S(6, c + 1), gm1, g.delta);
        roe_mean_vjp<DIR>(R, gm1, g.delta, du6, Db, vbar, Hbar);
        pin(vbar[0]), pin(vbar[1]), pin(vbar[2]), pin(Hbar);
        adj_stage_fence();
        states(c, a, b);
#pragma unroll
        for (int v = 0; v < 5; ++v) ab[v] = bb[v] = 0.0;
        roe_cells_vjp(R, a, S(6, c), b, S(6, c + 1), gm1, vbar, Hbar, ab, bb);
    };
    // J^T f + us of cell c
    auto finish = [&](int c, double out[5]) {
        double w[5], fb[5];
        fb[0] = 0.0;
#pragma unroll
        for (int v = 0; v < 5; ++v) {
            w[v] = S(v, c), out[v] = A(v, c);
            if (v > 0) fb[v] = A(4 + v, c);
        }
        euler_flux_vjp<DIR>(w, gm1, fb, out);
    };
    int I = s0;
    if (ok) {
        double w[5], r[5];
        load5(u, cell(s0 - 2 + ta), w);
        load5(rbar, cell(s0 - 2 + ta), r);
        keep(ta, w, r);
        if (ta < NC - TA) {
            load5(u, cell(s0 - 2 + TA + ta), w);
            load5(rbar, cell(s0 - 2 + TA + ta), r);
            keep(TA + ta, w, r);
        }
#pragma unroll
        for (int v = 0; v < 9; ++v) {
            A(v, ta) = 0.0;
            if (ta < KA - TA) A(v, TA + ta) = 0.0;
        }
    }
    adj_stage_fence();
    if (ok && ta == 0) {  // dub of the left face of cell s0
        double H[5], dub[5];
#pragma unroll
        for (int v = 0; v < 5; ++v) H[v] = (S(7 + v, 2) - S(7 + v, 1)) * ih12;
        jump_adjoint(1, H, dub);
#pragma unroll
        for (int v = 0; v < 5; ++v) D(v, 0) = dub[v], UL(v, 0) = 0.0;
    }
    // the segments of a wave may differ by one cell, and so by one chunk
    for (bool live = ok; __any(live);) {
        adj_stage_fence();
        const bool act = live && I + ta < (SPARE ? s1 + 1 : s1), more = live && I + TA < s1;
        const double own = !SPARE || I + ta < s1 ? 1.0 : 0.0;
        double un[5], rn[5];
        if (more) {
            load5(u, cell(I + TA + 3 + ta), un);
            load5(rbar, cell(I + TA + 3 + ta), rn);
        }
        if (act) {
            // cell j = I + ta is staged cell ta + 2; its stencil starts at ta
            double Hl[5], Hr[5], x[5], xn[5], xb[5], L6, R6, dub[5], du[5];
#pragma unroll
            for (int v = 0; v < 5; ++v) {
                const double r0 = S(7 + v, ta + 2);
                Hl[v] = (r0 - S(7 + v, ta + 1)) * ih12;
                Hr[v] = own * ((S(7 + v, ta + 3) - r0) * ih12);
                pin(Hl[v]), pin(Hr[v]);
            }
            {
                double vn[5], p[5];
#pragma unroll
                for (int m = 0; m < 5; ++m) vn[m] = S(5, ta + m), p[m] = S(6, ta + m), xn[m] = S(1, ta + m);
#pragma unroll
                for (int v = 1; v < 5; ++v) {
#pragma unroll
                    for (int m = 0; m < 5; ++m) {
                        x[m] = xn[m] * vn[m];
                        if (v == 1 + DIR) x[m] += p[m];
                        if (v == 4) x[m] += p[m] * vn[m];
                        if (v < 4) xn[m] = S(v + 1, ta + m);
                    }
                    adj_stage_fence();
                    weno5_cell_vjp<WW>(x, eps4, Hr[v], own * Hl[v], xb, L6, R6);
#pragma unroll
                    for (int m = 0; m < 5; ++m) atomicAdd(&A(4 + v, ta + m), xb[m]);
                    adj_stage_fence();
                }
            }
            jump_adjoint(ta + 2, Hr, dub);
#pragma unroll
            for (int v = 0; v < 5; ++v) D(v, ta + 1) = dub[v], pin(dub[v]);
            adj_stage_fence();
            double dl = D(0, ta);
#pragma unroll
            for (int m = 0; m < 5; ++m) xn[m] = S(0, ta + m);
#pragma unroll
            for (int v = 0; v < 5; ++v) {
#pragma unroll
                for (int m = 0; m < 5; ++m) x[m] = xn[m];
                double Lb = -dub[v], Rb = own * dl;
                if (v == 1 + DIR) Lb += Hr[0], Rb += own * Hl[0];
                if (v < 4) {
#pragma unroll
                    for (int m = 0; m < 5; ++m) xn[m] = S(v + 1, ta + m);
                    dl = D(v + 1, ta);
                }
                adj_stage_fence();
                weno5_cell_vjp<WW>(x, eps4, Lb, Rb, xb, L6, R6);
                UL(v, ta + 1) = L6;
                du[v] = R6;
                pin(du[v]);
#pragma unroll
                for (int m = 0; m < 5; ++m) atomicAdd(&A(v, ta + m), xb[m]);
                adj_stage_fence();
            }
            // the left face; the first one of a segment is the neighbour's
            const double h = I + ta > s0 ? -1.0 : 0.0;
            double Db[5], ab[5], bb[5];
#pragma unroll
            for (int v = 0; v < 5; ++v) du[v] -= UL(v, ta), Db[v] = h * Hl[v];
            state_adjoint(ta + 1, Db, du, ab, bb);
#pragma unroll
            for (int v = 0; v < 5; ++v) {
                atomicAdd(&A(v, ta + 1), ab[v]);
                atomicAdd(&A(v, ta + 2), bb[v]);
            }
        }
        adj_stage_fence();
        if (live && I - 2 + ta <= s1 - 3) {
            const uint32_t q = cell(I - 2 + ta);
            double out[5], old[5];
            if (DIR != 0) load5(ubar, q, old);
            finish(ta, out);
#pragma unroll
            for (int v = 0; v < 5; ++v) *elem(ubar, n3, v, q) = DIR != 0 ? old[v] + out[v] : out[v];
        }
        adj_stage_fence();
        if (more) {
            // the last four sums, the last five staged cells and the last face go first
#pragma unroll
            for (int v = 0; v < 9; ++v) {
                const double a = ta < KA - TA ? A(v, TA + ta) : 0.0;
                A(v, ta) = a;
                if (ta < KA - TA) A(v, TA + ta) = 0.0;
            }
            if (ta < NC - TA) {
#pragma unroll
                for (int v = 0; v < 12; ++v) S(v, ta) = S(v, TA + ta);
            }
            if (ta == 0) {
#pragma unroll
                for (int v = 0; v < 5; ++v) D(v, 0) = D(v, TA), UL(v, 0) = UL(v, TA);
            }
            adj_stage_fence();
            keep(NC - TA + ta, un, rn);
            I += TA;
        }
        live = more;
    }
    adj_stage_fence();
    const int c1 = s1 - I;  // staged and summed cell of cell s1-2
    if (ok && ta == 0 && (!SPARE || c1 == TA)) {  // the last face
        double du[5], Db[5], ab[5], bb[5];
#pragma unroll
        for (int v = 0; v < 5; ++v) {
            double x[5], xb[5], L6, R6;
#pragma unroll
            for (int m = 0; m < 5; ++m) x[m] = S(v, c1 + m);
            weno5_cell_vjp<WW>(x, eps4, 0.0, 0.0, xb, L6, R6);
            du[v] = R6 - UL(v, c1);
            Db[v] = (S(7 + v, c1 + 1) - S(7 + v, c1 + 2)) * ih12;
        }
        state_adjoint(c1 + 1, Db, du, ab, bb);
#pragma unroll
        for (int v = 0; v < 5; ++v) {
            A(v, c1 + 1) += ab[v];
            A(v, c1 + 2) += bb[v];
        }
    }
    __syncthreads();
    if (ok && ta < 4) {
        const uint32_t q = cell(s1 - 2 + ta);
        double old[5], out[5];
        load5(ubar, q, old);
        finish(c1 + ta, out);
#pragma unroll
        for (int v = 0; v < 5; ++v) *elem(ubar, n3, v, q) = old[v] + out[v];
    }
}

// ---------------------------------------------------------------------------
// Viscous adjoint in one pass.  With Gbar_d = -D_d rbar (rows 1-4: momentum x, y, z and
// energy) the viscous fluxes give at every point
//   the stencil fields f_d, the adjoints that the transposed gradients D_d carry back:
//     f_x = (gxx, gxy, gxz, kappa E_x), f_y = (gxy, gyy, gyz, kappa E_y),
//     f_z = (gxz, gyz, gzz, kappa E_z), linear in Gbar with the point velocity as
//     coefficient (tau is symmetric: nine distinct values);
//   the point fields pa, the adjoints of the point velocities in the energy fluxes;
// and Wbar = pa - sum_d D_d f_d for W = (u, v, w, T), which the primitive map takes to
// ubar.  A block owns a 32 x 8 (x, y) tile and marches along z.  Per plane it forms f_x
// on the tile and its +-2 x halo and f_y on the tile and its +-2 y halo, from rbar
// staged in LDS with the +-4 halo these need and from the z derivatives of rbar at
// those points (register rings of five planes for the tile's columns, an LDS ring for
// the halo points), and f_z on the tile, whose z difference is applied two planes
// later from a register ring: the fields never go through memory.
// ---------------------------------------------------------------------------
constexpr int kAvTX = kViscTX, kAvTY = kViscTY;
constexpr int kAvRX = kAvTX + 8, kAvRY = kAvTY + 8;    // rbar box, origin (x0-4, y0-4)
constexpr int kAvHalo = 4 * kAvTY + 4 * kAvTX;         // x-halo then y-halo points of the tile
constexpr int kAvExt = 16 + 4 * kAvTY + 4 * kAvTX;     // further rbar points: corners, x and y extensions
static_assert(kAvHalo <= kPointThreads && kAvExt <= kPointThreads && kAvTX * kAvTY == kPointThreads, "tile");

// position in the rbar box of halo point h (x-halo: columns x0-2, x0-1, x0+TX, x0+TX+1
// of the tile's rows; y-halo: rows y0-2, y0-1, y0+TY, y0+TY+1 of the tile's columns)
__device__ __forceinline__ void av_halo_pos(int h, int &bx, int &by) {
    if (h < 4 * kAvTY) {
        const int c = h & 3;
        bx = c < 2 ? 2 + c : kAvTX + 2 + c;
        by = 4 + (h >> 2);
    } else {
        const int q = h - 4 * kAvTY, r = q / kAvTX;
        bx = 4 + q % kAvTX;
        by = r < 2 ? 2 + r : kAvTY + 2 + r;
    }
}
// position in the rbar box of further point e: the 2 x 2 corners between the halos,
// then columns x0-4, x0-3, x0+TX+2, x0+TX+3 of the tile's rows, then rows y0-4, y0-3,
// y0+TY+2, y0+TY+3 of its columns
__device__ __forceinline__ void av_ext_pos(int e, int &bx, int &by) {
    if (e < 16) {
        const int cc = e >> 2;
        bx = (cc & 1 ? kAvTX + 4 : 2) + (e & 1);
        by = (cc & 2 ? kAvTY + 4 : 2) + ((e >> 1) & 1);
    } else if (e < 16 + 4 * kAvTY) {
        const int q = e - 16, c = q & 3;
        bx = c < 2 ? c : kAvTX + 4 + c;
        by = 4 + (q >> 2);
    } else {
        const int q = e - 16 - 4 * kAvTY, r = q / kAvTX;
        bx = 4 + q % kAvTX;
        by = r < 2 ? r : kAvTY + 4 + r;
    }
}

// the fields of a point from its rbar gradient (Gbar[d][c] = -D_d rbar_c) and velocity
struct AvFields {
    double gxx, gyy, gzz, gxy, gxz, gyz, ex, ey, ez;
};
__device__ __forceinline__ AvFields av_fields(const double Gbar[3][4], const double v[3], double mu, double kc) {
    const double Ex = Gbar[0][3], Ey = Gbar[1][3], Ez = Gbar[2][3];
    const double bxx = Gbar[0][0] + Ex * v[0];
    const double byy = Gbar[1][1] + Ey * v[1];
    const double bzz = Gbar[2][2] + Ez * v[2];
    const double bxy = Gbar[0][1] + Gbar[1][0] + Ex * v[1] + Ey * v[0];
    const double bxz = Gbar[0][2] + Gbar[2][0] + Ex * v[2] + Ez * v[0];
    const double byz = Gbar[1][2] + Gbar[2][1] + Ey * v[2] + Ez * v[1];
    // tau_aa = mu (2 g_aa - 2/3 div), tau_ab = mu (g_ab + g_ba)
    const double divb = -2.0 / 3.0 * mu * (bxx + byy + bzz);
    AvFields f;
    f.gxx = 2.0 * mu * bxx + divb;
    f.gyy = 2.0 * mu * byy + divb;
    f.gzz = 2.0 * mu * bzz + divb;
    f.gxy = mu * bxy;
    f.gxz = mu * bxz;
    f.gyz = mu * byz;
    f.ex = kc * Ex;
    f.ey = kc * Ey;
    f.ez = kc * Ez;
    return f;
}

__global__ __launch_bounds__(kPointThreads, 2) void k_adj_visc(AdjGeom g, const double *__restrict__ u,
                                                               const double *__restrict__ rbar,
                                                               double *__restrict__ ubar, AdjEpilogue ep,
                                                               int zp) {
    constexpr int TX = kAvTX, TY = kAvTY, RX = kAvRX, RY = kAvRY;
    __shared__ double sR[4][RY][RX];             // rbar rows 1-4 of the plane
    __shared__ double sV[3][TY + 4][TX + 4];     // velocity of the plane, tile and +-2 halo
    __shared__ double sFx[4][TY][TX + 4];        // f_x, tile rows, x halo
    __shared__ double sFy[4][TY + 4][TX];        // f_y, tile columns, y halo
    __shared__ double hR[5][4][kAvHalo];         // rbar of the halo points, slot (plane - z0 + 4) mod 5
    const int nx = g.nx, ny = g.ny, nz = g.nz;
    const size_t n3 = g.n3, sz = (size_t)nx * ny;
    const int ntx = (nx + TX - 1) / TX, nty = (ny + TY - 1) / TY;
    const long long lb = blockIdx.x;
    const int x0 = (int)(lb % ntx) * TX, y0 = (int)((lb / ntx) % nty) * TY;
    const int z0 = (int)(lb / ((long long)ntx * nty)) * zp, z1 = min(z0 + zp, nz);
    const int t = threadIdx.x, tx = t % TX, ty = t / TX;
    const bool act = x0 + tx < nx && y0 + ty < ny;
    // a column past a ragged edge wraps periodically: its values are halo values of the
    // active columns beside it
    const size_t col = (size_t)wrapn(y0 + ty, ny) * nx + wrapn(x0 + tx, nx);
    const bool own_h = t < kAvHalo, own_e = t < kAvExt;
    int hbx = 0, hby = 0, ebx = 0, eby = 0;
    if (own_h) av_halo_pos(t, hbx, hby);
    if (own_e) av_ext_pos(t, ebx, eby);
    const size_t hcol = (size_t)wrapn(y0 - 4 + hby, ny) * nx + wrapn(x0 - 4 + hbx, nx);
    const size_t ecol = (size_t)wrapn(y0 - 4 + eby, ny) * nx + wrapn(x0 - 4 + ebx, nx);
    const double *rb = rbar + n3;  // rows 1..4
    const double mu = g.mu, kc = g.mu / ((g.gamma - 1.0) * g.prandtl), gm1 = g.gamma - 1.0;
    const double ihx = g.ih[0], ihy = g.ih[1], ihz = g.ih[2];
    auto slot = [&](int p) { return (p - z0 + 4) % 5; };
    auto vel_at = [&](size_t i, double v[3]) {
        const double inv = rcp(u[i]);
        v[0] = u[n3 + i] * inv;
        v[1] = u[2 * n3 + i] * inv;
        v[2] = u[3 * n3 + i] * inv;
    };
    double Rz[5][4];  // rbar of this column at planes k-2 .. k+2
    double Vz[5][3];  // velocity of this column at planes k-2 .. k+2
    // Wbar of this column at planes k-2 .. k+2 as it accumulates: pa - D_x f_x - D_y f_y
    // when its plane is formed, and the terms of -D_z f_z as the f_z of the planes two
    // on either side are formed (the plane k-2 is complete after plane k)
    double Tq[5][4];
    const int k0 = z0 - 2;
    auto is_full = [&](int k) { return k >= z0 && k < z1; };
#pragma unroll
    for (int m = 0; m < 5; ++m) {
        const size_t q = col + (size_t)wrapn(k0 - 2 + m, nz) * sz;
#pragma unroll
        for (int c = 0; c < 4; ++c) Rz[m][c] = rb[c * n3 + q];
        vel_at(q, Vz[m]);
        if (own_h) {
            const size_t qh = hcol + (size_t)wrapn(k0 - 2 + m, nz) * sz;
#pragma unroll
            for (int c = 0; c < 4; ++c) hR[slot(k0 - 2 + m)][c][t] = rb[c * n3 + qh];
        }
    }
#pragma unroll
    for (int m = 0; m < 5; ++m)
#pragma unroll
        for (int c = 0; c < 4; ++c) Tq[m][c] = 0.0;
    const double cz = ihz * (1.0 / 12.0);
    // loads for the plane after the current one (halo velocities, further rbar points)
    double hu[4] = {1.0, 0.0, 0.0, 0.0}, er[4] = {0.0, 0.0, 0.0, 0.0};
    for (int k = k0; k < z1 + 2; ++k) {
        // planes z0 .. z1-1 are formed in full; the two planes on either side only for f_z.
        // Every load is issued one iteration (the rings three planes) ahead of its use.
        const bool full = is_full(k);
        double Rn[4], Un[4], Hn[4];  // plane k+3 of the column and of the halo point
        {
            const size_t q = col + (size_t)wrapn(k + 3, nz) * sz;
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                Rn[c] = rb[c * n3 + q];
                Un[c] = u[c * n3 + q];
            }
            if (own_h) {
                const size_t qh = hcol + (size_t)wrapn(k + 3, nz) * sz;
#pragma unroll
                for (int c = 0; c < 4; ++c) Hn[c] = rb[c * n3 + qh];
            }
        }
        const int ko = k - 2;  // finished in this iteration: its f_z are known two planes on either side
        const bool out = ko >= z0 && act;
        const size_t po = (size_t)wrapn(ko, nz) * sz + col;
        double us[5], ubv[5];
        if (out) {
#pragma unroll
            for (int v = 0; v < 5; ++v) {
                us[v] = u[v * n3 + po];
                ubv[v] = ubar[v * n3 + po];
            }
        }
        if (own_h) {
            const int s0 = slot(k);
#pragma unroll
            for (int c = 0; c < 4; ++c) sR[c][hby][hbx] = hR[s0][c][t];
            if (full) {
                const double inv = rcp(hu[0]);
#pragma unroll
                for (int c = 0; c < 3; ++c) sV[c][hby - 2][hbx - 2] = hu[1 + c] * inv;
            }
        }
        if (own_e && full) {
#pragma unroll
            for (int c = 0; c < 4; ++c) sR[c][eby][ebx] = er[c];
        }
        if (is_full(k + 1)) {
            if (own_h) {
                const size_t qh = hcol + (size_t)wrapn(k + 1, nz) * sz;
#pragma unroll
                for (int c = 0; c < 4; ++c) hu[c] = u[c * n3 + qh];
            }
            if (own_e) {
                const size_t qe = ecol + (size_t)wrapn(k + 1, nz) * sz;
#pragma unroll
                for (int c = 0; c < 4; ++c) er[c] = rb[c * n3 + qe];
            }
        }
#pragma unroll
        for (int c = 0; c < 4; ++c) sR[c][ty + 4][tx + 4] = Rz[2][c];
#pragma unroll
        for (int c = 0; c < 3; ++c) sV[c][ty + 2][tx + 2] = Vz[2][c];
        __syncthreads();
        double pa[3] = {0.0, 0.0, 0.0};
        {
            // the tile's point: rbar gradient, fields
            const int X = tx + 4, Y = ty + 4;
            double Gbar[3][4];
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                Gbar[0][c] = -dcen(sR[c][Y][X - 2], sR[c][Y][X - 1], sR[c][Y][X + 1], sR[c][Y][X + 2]) * ihx;
                Gbar[1][c] = -dcen(sR[c][Y - 2][X], sR[c][Y - 1][X], sR[c][Y + 1][X], sR[c][Y + 2][X]) * ihy;
                Gbar[2][c] = -dcen(Rz[0][c], Rz[1][c], Rz[3][c], Rz[4][c]) * ihz;
            }
            const AvFields f = av_fields(Gbar, Vz[2], mu, kc);
            // -D_z f_z: dcen(m2, m1, p1, p2) = (8 (p1 - m1) - (p2 - m2)) / 12, so f_z of this
            // plane enters the planes k+2, k+1, k-1, k-2 with -1, 8, -8, 1 times cz
            const double fz[4] = {f.gxz, f.gyz, f.gzz, f.ez};
#pragma unroll
            for (int a = 0; a < 4; ++a) {
                const double w = cz * fz[a];
                Tq[4][a] = -w;
                Tq[3][a] += 8.0 * w;
                Tq[1][a] -= 8.0 * w;
                Tq[0][a] += w;
            }
            if (full) {
                sFx[0][ty][tx + 2] = f.gxx;
                sFx[1][ty][tx + 2] = f.gxy;
                sFx[2][ty][tx + 2] = f.gxz;
                sFx[3][ty][tx + 2] = f.ex;
                sFy[0][ty + 2][tx] = f.gxy;
                sFy[1][ty + 2][tx] = f.gyy;
                sFy[2][ty + 2][tx] = f.gyz;
                sFy[3][ty + 2][tx] = f.ey;
                // point fields: the velocity gradients of the plane, tau
                double gv[3][3];  // gv[a][b] = d v_a / d x_b
#pragma unroll
                for (int a = 0; a < 3; ++a) {
                    gv[a][0] = dcen(sV[a][ty + 2][tx], sV[a][ty + 2][tx + 1], sV[a][ty + 2][tx + 3],
                                    sV[a][ty + 2][tx + 4]) * ihx;
                    gv[a][1] = dcen(sV[a][ty][tx + 2], sV[a][ty + 1][tx + 2], sV[a][ty + 3][tx + 2],
                                    sV[a][ty + 4][tx + 2]) * ihy;
                    gv[a][2] = dcen(Vz[0][a], Vz[1][a], Vz[3][a], Vz[4][a]) * ihz;
                }
                const double div = gv[0][0] + gv[1][1] + gv[2][2];
                const double tdiv = 2.0 / 3.0 * div;
                const double txx = mu * (2.0 * gv[0][0] - tdiv), tyy = mu * (2.0 * gv[1][1] - tdiv),
                             tzz = mu * (2.0 * gv[2][2] - tdiv);
                const double txy = mu * (gv[0][1] + gv[1][0]), txz = mu * (gv[0][2] + gv[2][0]),
                             tyz = mu * (gv[1][2] + gv[2][1]);
                const double Ex = Gbar[0][3], Ey = Gbar[1][3], Ez = Gbar[2][3];
                pa[0] = Ex * txx + Ey * txy + Ez * txz;
                pa[1] = Ex * txy + Ey * tyy + Ez * tyz;
                pa[2] = Ex * txz + Ey * tyz + Ez * tzz;
            }
        }
        if (own_h && full) {
            // a halo point: rbar gradient (z from the halo ring), its f_x or f_y
            double Gbar[3][4];
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                Gbar[0][c] = -dcen(sR[c][hby][hbx - 2], sR[c][hby][hbx - 1], sR[c][hby][hbx + 1],
                                   sR[c][hby][hbx + 2]) * ihx;
                Gbar[1][c] = -dcen(sR[c][hby - 2][hbx], sR[c][hby - 1][hbx], sR[c][hby + 1][hbx],
                                   sR[c][hby + 2][hbx]) * ihy;
                Gbar[2][c] = -dcen(hR[slot(k - 2)][c][t], hR[slot(k - 1)][c][t], hR[slot(k + 1)][c][t],
                                   hR[slot(k + 2)][c][t]) * ihz;
            }
            const double v[3] = {sV[0][hby - 2][hbx - 2], sV[1][hby - 2][hbx - 2], sV[2][hby - 2][hbx - 2]};
            const AvFields f = av_fields(Gbar, v, mu, kc);
            if (t < 4 * TY) {
                const int r = hby - 4, cx = hbx - 2;
                sFx[0][r][cx] = f.gxx;
                sFx[1][r][cx] = f.gxy;
                sFx[2][r][cx] = f.gxz;
                sFx[3][r][cx] = f.ex;
            } else {
                const int r = hby - 2, cx = hbx - 4;
                sFy[0][r][cx] = f.gxy;
                sFy[1][r][cx] = f.gyy;
                sFy[2][r][cx] = f.gyz;
                sFy[3][r][cx] = f.ey;
            }
        }
        __syncthreads();
        if (full) {
#pragma unroll
            for (int a = 0; a < 4; ++a) {
                double s = a < 3 ? pa[a] : 0.0;
                s -= dcen(sFx[a][ty][tx], sFx[a][ty][tx + 1], sFx[a][ty][tx + 3], sFx[a][ty][tx + 4]) * ihx;
                s -= dcen(sFy[a][ty][tx], sFy[a][ty + 1][tx], sFy[a][ty + 3][tx], sFy[a][ty + 4][tx]) * ihy;
                Tq[2][a] += s;
            }
        }
        if (out) {
            const double *Wb = Tq[0];
            // W = (m_k / rho, gamma p / rho), p = (gamma-1)(e - m.v/2)
            const double r = us[0], m[3] = {us[1], us[2], us[3]}, e = us[4];
            const double inv = rcp(r);
            const double v[3] = {m[0] * inv, m[1] * inv, m[2] * inv};
            const double qq = m[0] * v[0] + m[1] * v[1] + m[2] * v[2];
            const double pr = gm1 * (e - 0.5 * qq);
            // T = gamma pr inv
            const double prb = g.gamma * inv * Wb[3];
            double invb = g.gamma * pr * Wb[3];
            const double eb = gm1 * prb;
            const double qqb = -0.5 * gm1 * prb;
            double mb[3];
#pragma unroll
            for (int c = 0; c < 3; ++c) {
                const double vb = Wb[c] + qqb * m[c];
                mb[c] = qqb * v[c] + vb * inv;
                invb += vb * m[c];
            }
            const double fin[5] = {ubv[0] + -invb * inv * inv, ubv[1] + mb[0], ubv[2] + mb[1], ubv[3] + mb[2],
                                   ubv[4] + eb};
#pragma unroll
            for (int v = 0; v < 5; ++v) {
                const size_t o = v * n3 + po;
                if (ep.store_ub) ubar[o] = fin[v];
                adj_epilogue_at(ep, o, fin[v]);
            }
        }
        // advance the rings; plane k+3 enters them
#pragma unroll
        for (int m = 0; m < 4; ++m) {
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                Rz[m][c] = Rz[m + 1][c];
                Tq[m][c] = Tq[m + 1][c];
            }
#pragma unroll
            for (int c = 0; c < 3; ++c) Vz[m][c] = Vz[m + 1][c];
        }
        {
            const double inv = rcp(Un[0]);
#pragma unroll
            for (int c = 0; c < 4; ++c) Rz[4][c] = Rn[c];
#pragma unroll
            for (int c = 0; c < 3; ++c) Vz[4][c] = Un[1 + c] * inv;
        }
        if (own_h) {
            const int s3 = slot(k + 3);
#pragma unroll
            for (int c = 0; c < 4; ++c) hR[s3][c][t] = Hn[c];
        }
    }
}

// out = a x + b y (y may be null)
__global__ void k_lincomb(size_t n, double a, const double *__restrict__ x, double b, const double *__restrict__ y,
                          double *__restrict__ out) {
    const size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x;
    if (i >= n) return;
    out[i] = y ? a * x[i] + b * y[i] : a * x[i];
}

// out = x
__global__ void k_copy(size_t n, const double *__restrict__ x, double *__restrict__ out) {
    const size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x;
    if (i < n) out[i] = x[i];
}

// ubar = dK/du with K = <|m|^2 / (2 rho)>
__global__ void k_ke_seed(size_t n3, const double *__restrict__ u, double *__restrict__ ubar) {
    const size_t p = blockIdx.x * (size_t)blockDim.x + threadIdx.x;
    if (p >= n3) return;
    const double s = 1.0 / (double)n3;
    const double r = u[p], mx = u[n3 + p], my = u[2 * n3 + p], mz = u[3 * n3 + p];
    const double inv = 1.0 / r;
    ubar[p] = -0.5 * (mx * mx + my * my + mz * mz) * inv * inv * s;
    ubar[n3 + p] = mx * inv * s;
    ubar[2 * n3 + p] = my * inv * s;
    ubar[3 * n3 + p] = mz * inv * s;
    ubar[4 * n3 + p] = 0.0;
}

// vbar_i = rho (mbar_i + ebar v_i): the initial-state map u(rho, v, p) transposed at fixed rho, p
__global__ void k_ic_vjp(size_t n3, const double *__restrict__ rho, const double *__restrict__ vel,
                         const double *__restrict__ ubar, double *__restrict__ vbar) {
    const size_t p = blockIdx.x * (size_t)blockDim.x + threadIdx.x;
    if (p >= n3) return;
    const double r = rho[p], eb = ubar[4 * n3 + p];
#pragma unroll
    for (int c = 0; c < 3; ++c) vbar[c * n3 + p] = r * (ubar[(1 + c) * n3 + p] + eb * vel[c * n3 + p]);
}

// ----------------------------------------------------------------------------
// launchers
// ----------------------------------------------------------------------------
static inline dim3 grid1(size_t n) { return dim3((unsigned)((n + 255) / 256)); }

// Lines and segments per block of k_adj_march (their product is at most the block).  The
// busiest CU decides: of its blocks two run side by side, one alone takes about 0.7 of the
// two's time, and a segment adds 0.4 steps of its own to its cells.  So small boxes get
// short segments on every CU, and ragged ones a split that leaves no nearly empty round.
struct MarchSplit {
    int Lb, nseg;
};
static MarchSplit march_split(size_t nlines, int n) {
    MarchSplit best{64, 1};
    double cost = 0.0;
    for (int Lb = 64; Lb >= 8; --Lb) {
        const int nseg = std::min(kAmThreads / Lb, n / 4);
        const size_t k = ((nlines + Lb - 1) / Lb + 255) / 256;
        const double c = (double)((n + nseg - 1) / nseg + 0.4) * ((double)(k / 2) * 2.0 + (k % 2 ? 1.4 : 0.0));
        if (Lb == 64 || c < cost) best = MarchSplit{Lb, nseg}, cost = c;
    }
    return best;
}

// Segments per line of k_adj_cells by the same estimate, in chunks of 16 cells
static int cells_split(size_t nlines, int n) {
    auto rounds = [&](int nseg) {
        const size_t lb = kAcSeg / nseg;
        return ((nlines + lb - 1) / lb + 255) / 256;
    };
    int best = 1;
    double cost = 0.0;
    for (int nseg = 1; nseg <= kAcSeg && nseg <= n / 4; nseg *= 2) {
        const size_t k = rounds(nseg);
        const int len = (n + nseg - 1) / nseg;
        const double c = ((len + kAcTA - 1) / kAcTA + 0.4) * ((double)(k / 2) * 2.0 + (k % 2 ? 1.4 : 0.0));
        if (nseg == 1 || c < cost) best = nseg, cost = c;
    }
    // a segment of full chunks has no spare lane for its last face: halved where that takes no
    // further round
    const int twice = 2 * best;
    if (twice <= kAcSeg && twice <= n / 4 && (n + best - 1) / best % kAcTA == 0 && rounds(twice) == rounds(best)) best = twice;
    return best;
}

template <int WW>
static void adj_conv(const BoxDesc &b, hipStream_t s, const AdjGeom &g, const double *u, const double *rbar,
                     double *ubar) {
    const size_t lx = (size_t)b.ny * b.nz, ly = (size_t)b.nx * b.nz, lz = (size_t)b.nx * b.ny;
    // The march fills the chip from about 64^3 points on (32 us along y there, 128^3 167); below,
    // its shortest segments of four cells in turn take longer than a chunk of cells side by side
    // (32^3: 24.4 us against 13.0).
    const bool small = b.n3 < (1u << 18);
    auto cells = [&](auto kernel, auto spare, size_t nlines, int n) {
        const int nseg = cells_split(nlines, n), lb = kAcSeg / nseg;
        const bool idle = n / nseg % kAcTA != 0 && (n + nseg - 1) / nseg % kAcTA != 0;  // in every segment's last chunk
        hipLaunchKernelGGL((small && idle ? spare : kernel), dim3((unsigned)((nlines + lb - 1) / lb)), dim3(256), 0, s, g, u,
                           rbar, ubar, nseg);
    };
    auto march = [&](auto kernel, size_t nlines, int n) {
        const MarchSplit m = march_split(nlines, n);
        hipLaunchKernelGGL(kernel, dim3((unsigned)((nlines + m.Lb - 1) / m.Lb)), dim3(kAmThreads), 0, s, g, u, rbar, ubar,
                           m.Lb, m.nseg);
    };
    cells(k_adj_cells<0, WW, false>, k_adj_cells<0, WW, true>, lx, b.nx);
    if (small) {
        cells(k_adj_cells<1, WW, false>, k_adj_cells<1, WW, true>, ly, b.ny);
        cells(k_adj_cells<2, WW, false>, k_adj_cells<2, WW, true>, lz, b.nz);
    } else {
        march(k_adj_march<1, WW>, ly, b.ny);
        march(k_adj_march<2, WW>, lz, b.nz);
    }
}

// the stage-combination epilogue by separate launches (boxes without viscous terms)
__global__ void k_epilogue(size_t n, const double *__restrict__ fin, AdjEpilogue e) {
    const size_t o = blockIdx.x * (size_t)blockDim.x + threadIdx.x;
    if (o >= n) return;
    adj_epilogue_at(e, o, fin[o]);
}

// Planes per block of k_adj_visc: a block forms two planes of lookahead on either side again,
// so it takes as many planes as leave a block for every CU (product of a 130 x 90 x 66 box:
// 315 us with 16 planes and 300 blocks, 341 with 4, 370 with 32; 32^3: 58 us with 2, 110 with
// 16), and 32 where that still leaves two (140^3: 2 % less than with 16).
static int adj_visc_planes(long long cols, int nz) {
    int zp = 32;
    while (zp > 2 && cols * ((nz + zp - 1) / zp) < (zp == 32 ? 512 : 256)) zp /= 2;
    return zp;
}

static void rhs_vjp(const BoxDesc &b, int weights, hipStream_t s, const double *u, const double *rbar, double *ubar,
                    const AdjEpilogue *epi) {
    const AdjGeom g = adj_geom(b);
    if (weights == CNS_WENO_Z) adj_conv<CNS_WENO_Z>(b, s, g, u, rbar, ubar);
    else if (weights == CNS_WENO_M) adj_conv<CNS_WENO_M>(b, s, g, u, rbar, ubar);
    else adj_conv<CNS_WENO_JS>(b, s, g, u, rbar, ubar);
    AdjEpilogue e;
    if (epi) e = *epi;
    if (b.mu > 0.0) {
        const long long cols = (long long)((b.nx + kAvTX - 1) / kAvTX) * ((b.ny + kAvTY - 1) / kAvTY);
        const int zp = adj_visc_planes(cols, b.nz);
        hipLaunchKernelGGL(k_adj_visc, dim3((unsigned)(cols * ((b.nz + zp - 1) / zp))), dim3(kPointThreads), 0, s, g, u, rbar,
                           ubar, e, zp);
    } else if (epi) {
        // ubar holds the finished product; the epilogue reads it from there
        const size_t n5 = 5 * b.n3;
        hipLaunchKernelGGL(k_epilogue, dim3((unsigned)((n5 + 255) / 256)), dim3(256), 0, s, n5, (const double *)ubar, e);
    }
}

void adj_rhs_vjp(const BoxDesc &b, int weights, hipStream_t s, const double *u, const double *rbar, double *ubar) {
    rhs_vjp(b, weights, s, u, rbar, ubar, nullptr);
}

void adj_rhs_vjp_epi(const BoxDesc &b, int weights, hipStream_t s, const double *u, const double *rbar, double *ubar,
                     const AdjEpilogue &epi) {
    rhs_vjp(b, weights, s, u, rbar, ubar, &epi);
}

void adj_lincomb(size_t n, double a, const double *x, double b, const double *y, double *out, hipStream_t s) {
    hipLaunchKernelGGL(k_lincomb, grid1(n), dim3(256), 0, s, n, a, x, b, y, out);
}
void adj_copy(size_t n, const double *x, double *out, hipStream_t s) {
    hipLaunchKernelGGL(k_copy, grid1(n), dim3(256), 0, s, n, x, out);
}
void adj_ke_seed(size_t n3, const double *u, double *ubar, hipStream_t s) {
    hipLaunchKernelGGL(k_ke_seed, grid1(n3), dim3(256), 0, s, n3, u, ubar);
}
void adj_ic_vjp(size_t n3, const double *rho, const double *vel, const double *ubar, double *vbar, hipStream_t s) {
    hipLaunchKernelGGL(k_ic_vjp, grid1(n3), dim3(256), 0, s, n3, rho, vel, ubar, vbar);
}

}  // namespace cns
