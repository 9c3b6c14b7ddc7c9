// cns_spectrum.hip -- kinetic-energy spectrum E(k) of a state on the GPU.
//
// The paper characterises its decaying-turbulence runs by the energy spectrum (Sec. 2.3:
// the model initial spectrum and the spectrum at t/tau = 3; Sec. 5: spectra per grid
// size) and by the Taylor microscale lambda behind Re_lambda and tau = lambda/u0.  Here
//   v_hat(k) = (1/N) sum_x v(x) exp(-i k.x),  N = nx ny nz,  v = m/rho,
//   E(k_s)   = sum over modes with round(|k|) = k_s of |v_hat|^2 / 2  (unit-width shells),
//   M2       = sum over all modes of |k|^2 |v_hat|^2 / 2,
// with the physical wavenumber k_d = 2 pi n_d / L_d.
//
// Steps (all on the plan's stream, FP64 whatever the plan's precision):
//   1. X1 = v_x + i v_y and X2 = v_z.  Two real fields share one complex transform: the
//      shells are symmetric under k -> -k, so sum_shell |X|^2 equals the sum of the two
//      real fields' |v_hat|^2 without separating them.  X2 is real, so only its
//      kx = 0 .. nx/2 are kept (the others count twice).
//   2. three launches of batched 1-D FFTs (x, then y, then z; each both fields) by a
//      mixed-radix Stockham autosort FFT (radix 8, 4, 2 and 3, 5, ... as generic small-prime
//      butterflies), the lines in LDS, or for powers of two along y and z in registers with LDS
//      for the exchanges between stages.  The x pass forms the velocities as it loads.  Each pass stores in the order in which the next one reads: W neighbouring
//      kx of all lines that a block takes next lie together, so the y and z passes read
//      contiguous runs (512^3: 64 KiB) and every store fills whole 128-byte lines.
//   3. the z pass does not store: it bins its modes.  A wave takes a line; along it the shell
//      grows with |kz|, so equal shells come in runs of neighbouring lanes: a segmented scan
//      (fixed doubling order) sums each run into its last lane, which adds it to the wave's
//      own histogram in LDS (the last lanes of one instruction hold different shells).
//      Fixed-order sums over the waves, over blocks and over shells follow: the result is the
//      same bits on every run.
// Scratch: the plan's stage buffers A, B (x pass), G (y pass), acc (twiddles), rhs (block
// partials).
//
// 512^3: 15.05 -> 5.0 ms (x 1.66, y 1.19, z with binning 2.20) against a floor of 0.9 ms (one
// read of density and momentum at the copy rate) and 3.7 ms for these passes' 17 GB; the z
// pass is bound by the LDS traffic and latency of the binning, one block of 8 waves on a CU.  Before: six passes of full complex
// fields in place, reading 64-byte pieces 8 KiB (y) and 4 MiB (z) apart at 2.1-2.6 TB/s, then
// 2.9 ms of binning by scans and ordered LDS additions.
#include <cmath>
#include <vector>

#include "cns_internal.h"

namespace cns {

constexpr int kFftPerThread = 8;  // elements a thread holds through a stage
constexpr int kFftMaxRadix = 32;
constexpr int kFftMaxW = 16;      // kx of a run
constexpr size_t kSpecLdsMax = 152 * 1024;

// Exact unsigned division by a divisor fixed at launch: q = (umulhi(n, M) + n) >> l with
// l = ceil(log2 d) and M = floor(2^32 (2^l - d) / d) + 1 (the round-up multiply-shift of
// Granlund and Montgomery), exact for every 32-bit n.
struct FastDiv {
    uint32_t M;
    int l;
};
static FastDiv fastdiv(uint32_t d) {
    int l = 0;
    while ((1ull << l) < d) ++l;
    return FastDiv{(uint32_t)((((1ull << 32) * ((1ull << l) - d)) / d) + 1), l};
}
__device__ __forceinline__ uint32_t fdiv(uint32_t n, FastDiv f) {
    return (uint32_t)(((uint64_t)__umulhi(n, f.M) + n) >> f.l);
}
// Division of small numbers: with M = ceil(2^32 / d), floor(n M / 2^32) = floor(n / d)
// whenever n < 2^16 and d < 2^16 (the error n (M d - 2^32) / (d 2^32) stays below 1/d).
// The in-line indexes of the stages (below 2^13) use it, with M formed on the device.
__device__ __forceinline__ uint64_t small_magic(uint32_t d) { return (uint64_t)(0xFFFFFFFFu / d) + 1u; }
__device__ __forceinline__ int sdiv(int n, uint64_t M) { return (int)(((uint64_t)(uint32_t)n * M) >> 32); }

// The same by a reciprocal in FP32, for a divisor known to the block: with n, d < 2^16 the
// rounding moves (n + 1/2) / d by less than its distance to the next integer.
__device__ __forceinline__ int qdiv(int n, float inv) { return (int)(((float)n + 0.5f) * inv); }

// the transform along one direction
struct FftPlan {
    int N;   // line length
    int nr;  // number of radix stages
    int radix[kFftMaxRadix];
    int ld;   // LDS stride between lines
    FastDiv dN;
    const double2 *tw;  // tw[k] = exp(-2 pi i k / N), k < N (global; each block copies it to LDS)
};

// LDS slots.  One slot in 17 of a line is left free and ld = 8 (mod 16), so that the strided
// stores of the first stages (8 j + s) and the loads of the y and z passes (l fastest)
// spread over all banks; one in 9 of the twiddles, which a stage reads at multiples of N / (8 Ns).
__host__ __device__ __forceinline__ int line_slots(int N) { return (N + N / 16 + 7) / 16 * 16 + 8; }
__host__ __device__ __forceinline__ int tw_slots(int N) { return N + N / 8 + 1; }
__device__ __forceinline__ int lds_at(int l, int j, const FftPlan &P) { return l * P.ld + j + (j >> 4); }
__device__ __forceinline__ int tw_at(int k) { return k + (k >> 3); }

__device__ __forceinline__ double2 cmul(double2 a, double2 b) {
    return make_double2(a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x);
}
__device__ __forceinline__ double2 cadd(double2 a, double2 b) { return make_double2(a.x + b.x, a.y + b.y); }
__device__ __forceinline__ double2 csub(double2 a, double2 b) { return make_double2(a.x - b.x, a.y - b.y); }

// DFTs of length 2, 4 and 8 in place
__device__ __forceinline__ void dft(double2 &a, double2 &b) {
    const double2 t = cadd(a, b);
    b = csub(a, b);
    a = t;
}
__device__ __forceinline__ void dft(double2 &a, double2 &b, double2 &c, double2 &d) {
    const double2 s0 = cadd(a, c), d0 = csub(a, c), s1 = cadd(b, d), d1 = csub(b, d);
    a = cadd(s0, s1);
    b = make_double2(d0.x + d1.y, d0.y - d1.x);  // d0 - i d1
    c = csub(s0, s1);
    d = make_double2(d0.x - d1.y, d0.y + d1.x);
}
__device__ __forceinline__ void dft8(double2 (&v)[8]) {
    constexpr double c = 0.70710678118654752440;
    double2 e[4] = {v[0], v[2], v[4], v[6]}, o[4] = {v[1], v[3], v[5], v[7]};
    dft(e[0], e[1], e[2], e[3]);
    dft(o[0], o[1], o[2], o[3]);
    o[1] = make_double2(c * (o[1].x + o[1].y), c * (o[1].y - o[1].x));   // times exp(-i pi/4)
    o[2] = make_double2(o[2].y, -o[2].x);                                // times -i
    o[3] = make_double2(c * (o[3].y - o[3].x), -c * (o[3].x + o[3].y));  // times exp(-3 i pi/4)
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        v[k] = cadd(e[k], o[k]);
        v[k + 4] = csub(e[k], o[k]);
    }
}

// One Stockham stage of radix R on nl lines of length N, in place in LDS: every thread
// reads the inputs of its butterflies into registers, the block synchronises, then the
// outputs are written.  Butterfly j (0 <= j < N/R) reads x[j + r N/R], r = 0..R-1,
// multiplies by the twiddles exp(-2 pi i r k/(Ns R)) with k = j mod Ns, takes a length-R
// DFT and writes output s to x[(j/Ns) Ns R + k + s Ns].
template <int R, int NT>
__device__ __forceinline__ void fft_stage_small(double2 *x, const double2 *tw, const FftPlan &P, int nl, int Ns) {
    const int N = P.N, m = N / R, tws = N / (Ns * R), nb = nl * m, tR = N / R;
    const uint64_t Mm = small_magic(m), Mns = small_magic(Ns);
    constexpr int NB = (kFftPerThread + R - 1) / R;
    double2 v[NB][R];
    int lo[NB], oo[NB];
#pragma unroll
    for (int q = 0; q < NB; ++q) {
        const int t = threadIdx.x + q * NT;
        if (t < nb) {
            const int l = sdiv(t, Mm), j = t - l * m;
            const int jn = sdiv(j, Mns), k = j - jn * Ns;
            lo[q] = l;
            oo[q] = jn * Ns * R + k;
#pragma unroll
            for (int r = 0; r < R; ++r) {
                v[q][r] = x[lds_at(l, j + r * m, P)];
                if (r && Ns > 1) v[q][r] = cmul(v[q][r], tw[tw_at(r * k * tws)]);
            }
        }
    }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < NB; ++q) {
        const int t = threadIdx.x + q * NT;
        if (t < nb) {
            const int l = lo[q], o = oo[q];
            if constexpr (R == 2) {
                x[lds_at(l, o, P)] = cadd(v[q][0], v[q][1]);
                x[lds_at(l, o + Ns, P)] = csub(v[q][0], v[q][1]);
            } else if constexpr (R == 8) {
                dft8(v[q]);
#pragma unroll
                for (int s = 0; s < 8; ++s) x[lds_at(l, o + s * Ns, P)] = v[q][s];
            } else if constexpr (R == 4) {
                dft(v[q][0], v[q][1], v[q][2], v[q][3]);
#pragma unroll
                for (int s = 0; s < 4; ++s) x[lds_at(l, o + s * Ns, P)] = v[q][s];
            } else {
#pragma unroll
                for (int s = 0; s < R; ++s) {
                    double2 acc = v[q][0];
#pragma unroll
                    for (int r = 1; r < R; ++r) acc = cadd(acc, cmul(v[q][r], tw[tw_at(((r * s) % R) * tR)]));
                    x[lds_at(l, o + s * Ns, P)] = acc;
                }
            }
        }
    }
    __syncthreads();
}

// generic radix R (any prime above 5): one work item per output, outputs held in
// registers until every input has been read.  Bound by the R products of an output and their
// LDS reads: with the two powers of the root in one product a spectrum of 257 x 64 x 64 takes
// 534 us, 800 with a product for each, of 16 x 16 x 1021 790 and 1096
template <int NT>
__device__ __forceinline__ void fft_stage_generic(double2 *x, const double2 *tw, const FftPlan &P, int nl, int Ns,
                                                  int R) {
    const int N = P.N, m = N / R, tws = N / (Ns * R);
    const uint64_t MN = small_magic(N), Mm = small_magic(m), Mns = small_magic(Ns);
    double2 out[kFftPerThread];
    int at[kFftPerThread];
#pragma unroll
    for (int q = 0; q < kFftPerThread; ++q) {
        const int t = threadIdx.x + q * NT;
        if (t < nl * N) {
            const int l = sdiv(t, MN), qq = t - l * N;
            const int s = sdiv(qq, Mm), j = qq - s * m;
            const int jn = sdiv(j, Mns), k = j - jn * Ns;
            // the twiddle exp(-2 pi i r k / (Ns R)) and the DFT's exp(-2 pi i r s / R) are one power
            const int dw = k * tws + s * m;
            double2 acc = x[lds_at(l, j, P)];
            int rw = 0;
            for (int r = 1; r < R; ++r) {
                rw += dw;
                if (rw >= N) rw -= N;
                acc = cadd(acc, cmul(x[lds_at(l, j + r * m, P)], tw[tw_at(rw)]));
            }
            out[q] = acc;
            at[q] = lds_at(l, jn * Ns * R + k + s * Ns, P);
        }
    }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < kFftPerThread; ++q) {
        const int t = threadIdx.x + q * NT;
        if (t < nl * N) x[at[q]] = out[q];
    }
    __syncthreads();
}

// all stages of nl lines staged in LDS (they end with a barrier).  POW2: only the radices 8, 4
// and 2 are compiled in (fewer registers than the odd radices bring).
template <bool POW2, int NT>
__device__ __forceinline__ void fft_lines(double2 *lines, const double2 *tw, const FftPlan &P, int nl) {
    __syncthreads();
    int Ns = 1;
    for (int st = 0; st < P.nr; ++st) {
        const int R = P.radix[st];
        if (R == 8) fft_stage_small<8, NT>(lines, tw, P, nl, Ns);
        else if (R == 4) fft_stage_small<4, NT>(lines, tw, P, nl, Ns);
        else if (R == 2) fft_stage_small<2, NT>(lines, tw, P, nl, Ns);
        else if constexpr (!POW2) {
            if (R == 3) fft_stage_small<3, NT>(lines, tw, P, nl, Ns);
            else if (R == 5) fft_stage_small<5, NT>(lines, tw, P, nl, Ns);
            else fft_stage_generic<NT>(lines, tw, P, nl, Ns, R);
        }
        Ns *= R;
    }
}

// The same transforms with the lines in registers, for lengths that are powers of two from 8
// on: the thread (l, tj) of N/8 per line holds elements tj + r N/8, which are the inputs of
// its radix-8 butterfly of the first stage; the lines go through LDS between stages only
// (512: twice, where staging every stage moves them four times), and the last stage's
// outputs stay in registers.  Element v[i] then has index out_index(i).
struct RegFft {
    int l, tj, m8, N, Rlast;
    bool act;
    __device__ __forceinline__ int out_index(int i) const {
        const int R = Rlast, q = i / R, s = i - q * R;
        return tj + q * m8 + s * (N / R);
    }
};
template <int R>
__device__ __forceinline__ void reg_stage(double2 (&v)[8], const double2 *x, const double2 *tw, const FftPlan &P,
                                          const RegFft &G, int Ns) {
    const int N = P.N, tws = N / (Ns * R);
#pragma unroll
    for (int q = 0; q < 8 / R; ++q) {
        const int j = G.tj + q * G.m8, k = j & (Ns - 1);
#pragma unroll
        for (int r = 0; r < R; ++r) {
            v[q * R + r] = x[lds_at(G.l, j + r * (N / R), P)];
            if (r) v[q * R + r] = cmul(v[q * R + r], tw[tw_at(r * k * tws)]);
        }
        if constexpr (R == 2) dft(v[2 * q], v[2 * q + 1]);
        else if constexpr (R == 4) dft(v[4 * q], v[4 * q + 1], v[4 * q + 2], v[4 * q + 3]);
        else dft8(v);
    }
}
template <int R>
__device__ __forceinline__ void reg_write(const double2 (&v)[8], double2 *x, const FftPlan &P, const RegFft &G, int Ns) {
#pragma unroll
    for (int q = 0; q < 8 / R; ++q) {
        const int j = G.tj + q * G.m8, k = j & (Ns - 1), o = (j - k) * R + k;
#pragma unroll
        for (int s = 0; s < R; ++s) x[lds_at(G.l, o + s * Ns, P)] = v[q * R + s];
    }
}
__device__ __forceinline__ void reg_fft(double2 (&v)[8], double2 *x, const double2 *tw, const FftPlan &P, RegFft &G) {
    if (G.act) dft8(v);
    if (P.nr > 1 && G.act) reg_write<8>(v, x, P, G, 1);
    int Ns = 8;
    G.Rlast = 8;
    for (int st = 1; st < P.nr; ++st) {
        // the radices are 8s, then at most one 4 or 2 (the last stage)
        const int rest = P.N / Ns;
        __syncthreads();
        if (rest >= 8) {
            if (G.act) reg_stage<8>(v, x, tw, P, G, Ns);
            if (rest > 8) {
                __syncthreads();
                if (G.act) reg_write<8>(v, x, P, G, Ns);
            }
        } else if (rest == 4) {
            if (G.act) reg_stage<4>(v, x, tw, P, G, Ns);
            G.Rlast = 4;
        } else {
            if (G.act) reg_stage<2>(v, x, tw, P, G, Ns);
            G.Rlast = 2;
        }
        Ns *= 8;
    }
}

// Order of the transformed fields.  A field holds nk kx (X1: nx, X2: nx/2 + 1), cut into runs
// of W (the last one shorter, w).  After the x pass element (kx, y, z) of run r lies at
// r sa + (z ny + y) w + (kx - r W): the (kx, y) of one z and run are contiguous, the lines of
// a block of the y pass.  After the y pass (kx, ky, z) lies at r sb + (ky (nz + pz) + z) w +
// (kx - r W): the lines of a block of the z pass.  In large boxes the strides over runs and
// ky are kept off powers of two, at which all pieces of a block's stores would meet in few
// memory channels.
struct SpecFields {
    int nx, ny, nz;
    int W;
    int nk[2], nrun[2];
    size_t sa, sb;         // elements from run to run
    int pz;
    double2 *a[2], *b[2];  // after the x and after the y pass
};

// the task of a block: blocks of one XCD take neighbouring tasks
__device__ __forceinline__ int task_of(int total) {
    const int b = blockIdx.x, x = b & 7, l = b >> 3;
    const int q = total >> 3, r = total & 7;
    return x * q + min(x, r) + l;  // l-th of range x
}

// x pass: the transforms of nl rows of both fields
template <typename T, bool POW2, int NT>
__global__ __launch_bounds__(NT) void k_fft_x(const T *u, size_t n3, FftPlan P, SpecFields F, int nl) {
    extern __shared__ double2 lds_c[];  // twiddles, then [nl][ld] lines
    double2 *tws = lds_c, *lines = lds_c + tw_slots(P.N);
    const int N = P.N, nrows = F.ny * F.nz, row0 = task_of((nrows + nl - 1) / nl) * nl, nact = min(nl, nrows - row0);
    const int ne = nact * N;
    for (int k = threadIdx.x; k < N; k += NT) tws[tw_at(k)] = P.tw[k];
    double vz[kFftPerThread];
    const size_t e0 = (size_t)row0 * N;
#pragma unroll
    for (int q = 0; q < kFftPerThread; ++q) {
        const int t = threadIdx.x + q * NT;
        vz[q] = 0.0;
        if (t < ne) {
            const int l = (int)fdiv(t, P.dN), j = t - l * N;
            const size_t e = e0 + t;
            const double ir = rcp(double(u[e]));
            lines[lds_at(l, j, P)] = make_double2(double(u[n3 + e]) * ir, double(u[2 * n3 + e]) * ir);
            vz[q] = double(u[3 * n3 + e]) * ir;
        }
    }
#pragma unroll
    for (int f = 0; f < 2; ++f) {
        if (f == 1) {
            __syncthreads();  // the first field has been stored
#pragma unroll
            for (int q = 0; q < kFftPerThread; ++q) {
                const int t = threadIdx.x + q * NT;
                if (t < ne) {
                    const int l = (int)fdiv(t, P.dN);
                    lines[lds_at(l, t - l * N, P)] = make_double2(vz[q], 0.0);
                }
            }
        }
        fft_lines<POW2, NT>(lines, tws, P, nl);
        // threads along (kx within a run, row, run): the rows of a run lie together
        const int W = F.W, nk = F.nk[f], full = nk / W;
        const float inw = 1.0f / (float)(nact * W), iw = 1.0f / (float)W, ilast = 1.0f / (float)max(nk - full * W, 1);
        for (int t = threadIdx.x; t < nact * nk; t += NT) {
            const int r = min(qdiv(t, inw), full), w = r < full ? W : nk - full * W;
            const int s = t - r * nact * W, l = qdiv(s, r < full ? iw : ilast), i = s - l * w;
            F.a[f][(size_t)r * F.sa + (size_t)(row0 + l) * w + i] = lines[lds_at(l, r * W + i, P)];
        }
    }
}

// y pass: a block transforms the lines of one z and run of one field.  POW2: in registers
template <bool POW2, int NT>
__global__ __launch_bounds__(NT) void k_fft_y(FftPlan P, SpecFields F) {
    extern __shared__ double2 lds_c[];
    double2 *tws = lds_c, *lines = lds_c + tw_slots(P.N);
    const int N = P.N, nz = F.nz;
    // tasks: z fastest, so that neighbouring blocks store neighbouring runs
    int task = task_of((F.nrun[0] + F.nrun[1]) * nz);
    const int f = task >= F.nrun[0] * nz ? 1 : 0;
    task -= f ? F.nrun[0] * nz : 0;
    const int r = task / nz, z = task - r * nz, w = min(F.W, (f ? F.nk[1] : F.nk[0]) - r * F.W);
    const double2 *src = (f ? F.a[1] : F.a[0]) + (size_t)r * F.sa + (size_t)z * N * w;
    double2 *dst = (f ? F.b[1] : F.b[0]) + (size_t)r * F.sb + (size_t)z * w;
    const size_t dk = (size_t)(nz + F.pz) * w;  // from ky to ky
    const int ne = w * N;
    const float iw = 1.0f / (float)w;
    double2 v[kFftPerThread];
    if constexpr (POW2) {
        RegFft G;
        G.N = N, G.m8 = N / 8;
        G.tj = qdiv(threadIdx.x, iw);
        G.l = threadIdx.x - G.tj * w;
        G.act = G.tj < G.m8;
        if (G.act)
#pragma unroll
            for (int q = 0; q < 8; ++q) v[q] = src[(G.tj + q * G.m8) * w + G.l];
        for (int k = threadIdx.x; k < N; k += NT) tws[tw_at(k)] = P.tw[k];
        reg_fft(v, lines, tws, P, G);
        if (G.act)
#pragma unroll
            for (int q = 0; q < 8; ++q) dst[(size_t)G.out_index(q) * dk + G.l] = v[q];
    } else {
        for (int k = threadIdx.x; k < N; k += NT) tws[tw_at(k)] = P.tw[k];
#pragma unroll
        for (int q = 0; q < kFftPerThread; ++q) {
            const int t = threadIdx.x + q * NT;
            if (t < ne) v[q] = src[t];
        }
#pragma unroll
        for (int q = 0; q < kFftPerThread; ++q) {
            const int t = threadIdx.x + q * NT;
            if (t < ne) {
                const int j = qdiv(t, iw);
                lines[lds_at(t - j * w, j, P)] = v[q];
            }
        }
        fft_lines<POW2, NT>(lines, tws, P, w);
        for (int t = threadIdx.x; t < ne; t += NT) {
            const int j = qdiv(t, iw), i = t - j * w;
            dst[(size_t)j * dk + i] = lines[lds_at(i, j, P)];
        }
    }
}

// tw[k] = exp(-2 pi i k / N), k < N, for the three lengths, one after the other
__global__ void k_fft_twiddles(double2 *tw, int nx, int ny, int nz) {
    const int d = blockIdx.x, N = d == 0 ? nx : (d == 1 ? ny : nz);
    double2 *t = tw + (d > 0 ? nx : 0) + (d > 1 ? ny : 0);
    for (int k = threadIdx.x; k < N; k += blockDim.x) {
        double s, c;
        sincospi(-2.0 * (double)k / (double)N, &s, &c);
        t[k] = make_double2(c, s);
    }
}

struct SpecGeom {
    int nx, ny, nz, nshell;
    size_t n3;
    double kux, kuy, kuz;  // 2 pi / L_d
    double norm;           // 1 / n3^2
    int nh;                // waves of a z block that bin, each with a histogram
};

__device__ __forceinline__ int signed_freq(int i, int n) { return i < (n + 1) / 2 ? i : i - n; }

// z pass: a block transforms the lines of one ky and run of one field at a time and bins their
// modes; the next task's loads are issued before the binning.  Every wave that bins keeps one
// histogram over the block's tasks, which the block adds up and writes once, with its
// share of the second moment, as ns + 1 partials.
__device__ __forceinline__ int shell_of(double k2, int nshell) { return min((int)floor(sqrt(k2) + 0.5), nshell - 1); }
template <bool POW2, int NT>
__global__ __launch_bounds__(NT, 2) void k_fft_z_bin(FftPlan P, SpecFields F, SpecGeom G, int ntask, double *part) {
    extern __shared__ double2 lds_c[];
    constexpr int NW = NT / 64;
    const int N = P.N, ns = G.nshell;
    double2 *tws = lds_c;                           // twiddles
    double2 *lines = tws + tw_slots(N);             // [W][ld] lines
    double *hist = (double *)(lines + F.W * P.ld);  // [nh][nshell]
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    double *hw = hist + (size_t)wv * ns;
    for (int k = threadIdx.x; k < N; k += NT) tws[tw_at(k)] = P.tw[k];
    for (int s = threadIdx.x; s < G.nh * ns; s += NT) hist[s] = 0.0;
    const int mh = N / 2;  // |kz| = 0 .. mh
    double m2 = 0.0;
    // consecutive tasks for the blocks of an XCD, a stride of their number for each
    const int nb = gridDim.x, X = min(nb, 8), x = blockIdx.x % X;
    const int q8 = ntask / X, r8 = ntask % X, lo = x * q8 + min(x, r8), hi = lo + q8 + (x < r8 ? 1 : 0);
    const int step = nb / X + (x < nb % X ? 1 : 0);
    double2 v[kFftPerThread];
    RegFft T;
    int f, r, iy, w;
    auto fetch = [&](int task) {
        f = task >= F.nrun[0] * F.ny ? 1 : 0;
        task -= f ? F.nrun[0] * F.ny : 0;
        r = task / F.ny;
        iy = task - r * F.ny;
        w = min(F.W, (f ? F.nk[1] : F.nk[0]) - r * F.W);
        const double2 *src = (f ? F.b[1] : F.b[0]) + (size_t)r * F.sb + (size_t)iy * (N + F.pz) * w;
        if constexpr (POW2) {
            T.N = N, T.m8 = N / 8;
            T.tj = qdiv(threadIdx.x, 1.0f / (float)w);
            T.l = threadIdx.x - T.tj * w;
            T.act = T.tj < T.m8;
            if (T.act)
#pragma unroll
                for (int q = 0; q < 8; ++q) v[q] = src[(T.tj + q * T.m8) * w + T.l];
        } else {
#pragma unroll
            for (int q = 0; q < kFftPerThread; ++q) {
                const int t = threadIdx.x + q * NT;
                if (t < w * N) v[q] = src[t];
            }
        }
    };
    int task = lo + (int)(blockIdx.x / X);
    if (task < hi) fetch(task);
    for (; task < hi; task += step) {
        const int f0 = f, x0 = r * F.W, nl = w;
        const double ky = signed_freq(iy, F.ny) * G.kuy;
        // the modes' |X|^2, mode kz of line l at l * ld + kz
        double *pw = (double *)lines;
        if constexpr (POW2) {
            reg_fft(v, lines, tws, P, T);
            __syncthreads();  // every thread has read the last exchange
            if (T.act)
#pragma unroll
                for (int q = 0; q < 8; ++q) pw[T.l * P.ld + T.out_index(q)] = v[q].x * v[q].x + v[q].y * v[q].y;
        } else {
            const float iw = 1.0f / (float)w;
#pragma unroll
            for (int q = 0; q < kFftPerThread; ++q) {
                const int t = threadIdx.x + q * NT;
                if (t < nl * N) {
                    const int j = qdiv(t, iw);
                    lines[lds_at(t - j * nl, j, P)] = v[q];
                }
            }
            fft_lines<POW2, NT>(lines, tws, P, nl);
#pragma unroll
            for (int q = 0; q < kFftPerThread; ++q) {
                const int t = threadIdx.x + q * NT;
                if (t < nl * N) {
                    const int j = qdiv(t, iw);
                    v[q] = lines[lds_at(t - j * nl, j, P)];
                }
            }
            __syncthreads();
#pragma unroll
            for (int q = 0; q < kFftPerThread; ++q) {
                const int t = threadIdx.x + q * NT;
                if (t < nl * N) {
                    const int j = qdiv(t, iw);
                    pw[(t - j * nl) * P.ld + j] = v[q].x * v[q].x + v[q].y * v[q].y;
                }
            }
        }
        __syncthreads();
        if (task + step < hi) fetch(task + step);
        for (int l = wv; wv < G.nh && l < nl; l += G.nh) {
            const int kx = x0 + l;
            const double kxp = signed_freq(kx, F.nx) * G.kux, kp = kxp * kxp + ky * ky;
            // X2 keeps kx = 0 .. nx/2: the others mirror the ones between
            const double wt = f0 == 1 && kx != 0 && 2 * kx != F.nx ? G.norm : 0.5 * G.norm;
            for (int m0 = 0; m0 <= mh; m0 += 64) {
                const int m = m0 + lane;
                int s = -1;  // past the line's end: a run of its own that adds nothing
                double p = 0.0;
                if (m <= mh) {
                    p = pw[l * P.ld + m];
                    if (m != 0 && 2 * m != N) p += pw[l * P.ld + N - m];
                    p *= wt;
                    const double kz = m * G.kuz, k2 = kp + kz * kz;
                    s = shell_of(k2, ns);
                    m2 += k2 * p;
                }
                // run heads and tails
                const int sp = __shfl_up(s, 1, 64), sn = __shfl_down(s, 1, 64);
                int h = (lane == 0 || sp != s) ? 1 : 0;
                const bool tail = lane == 63 || sn != s;
#pragma unroll
                for (int d = 1; d < 64; d <<= 1) {
                    const double pu = __shfl_up(p, d, 64);
                    const int hu = __shfl_up(h, d, 64);
                    if (lane >= d) {
                        if (!h) p += pu;
                        h |= hu;
                    }
                }
                if (tail && s >= 0) hw[s] += p;
            }
        }
        __syncthreads();  // the next task overwrites the lines
    }
    double *out = part + (size_t)blockIdx.x * (ns + 1);
    __syncthreads();
    for (int s = threadIdx.x; s < ns; s += NT) {
        double a = hist[s];
        for (int q = 1; q < G.nh; ++q) a += hist[(size_t)q * ns + s];
        out[s] = a;
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) m2 += __shfl_xor(m2, o, 64);
    __syncthreads();
    if (lane == 0) hist[wv] = m2;
    __syncthreads();
    if (threadIdx.x == 0) {
        double a = hist[0];
        for (int q = 1; q < NW; ++q) a += hist[q];
        out[ns] = a;
    }
}

// sum over the block partials in a fixed order: one block per shell (and one for the second
// moment), its threads striding over the partials, then a fixed-shape tree in LDS
__global__ __launch_bounds__(kPointThreads) void k_spec_final(const double *part, int nblocks, int nshell, double *E,
                                                              double *M2) {
    __shared__ double re[kPointThreads];
    const int s = blockIdx.x;
    double e = 0.0;
    for (int b = threadIdx.x; b < nblocks; b += blockDim.x) e += part[(size_t)b * (nshell + 1) + s];
    re[threadIdx.x] = e;
    __syncthreads();
    for (int w = blockDim.x / 2; w > 0; w >>= 1) {
        if ((int)threadIdx.x < w) re[threadIdx.x] += re[threadIdx.x + w];
        __syncthreads();
    }
    if (threadIdx.x == 0) *(s < nshell ? E + s : M2) = re[0];
}

// mom = {sum_s E[s], M2} and the Taylor microscale lambda = sqrt(5 sum E / M2) of isotropic
// turbulence (+inf for a uniform velocity); one block, a fixed-shape tree
__global__ __launch_bounds__(kPointThreads) void k_spec_mom(const double *E, const double *M2, int nshell, double *mom) {
    __shared__ double re[kPointThreads];
    double e = 0.0;
    for (int s = threadIdx.x; s < nshell; s += blockDim.x) e += E[s];
    re[threadIdx.x] = e;
    __syncthreads();
    for (int w = blockDim.x / 2; w > 0; w >>= 1) {
        if ((int)threadIdx.x < w) re[threadIdx.x] += re[threadIdx.x + w];
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        const double m = M2[0];
        mom[0] = re[0];
        mom[1] = m;
        mom[2] = m > 0.0 ? sqrt(5.0 * re[0] / m) : __builtin_inf();
    }
}

// ---------------------------------------------------------------------------
// host side
// ---------------------------------------------------------------------------
static int fft_factor(int n, int *radix) {
    int nr = 0;
    while (n % 8 == 0) radix[nr++] = 8, n /= 8;
    while (n % 4 == 0) radix[nr++] = 4, n /= 4;
    while (n % 2 == 0) radix[nr++] = 2, n /= 2;
    for (int p = 3; n > 1; p += 2)
        while (n % p == 0) radix[nr++] = p, n /= p;
    return nr;
}

int spectrum_shells(const BoxDesc &b) {
    const double kx = (b.nx / 2) * (2.0 * M_PI * b.inv_h[0] / b.nx);
    const double ky = (b.ny / 2) * (2.0 * M_PI * b.inv_h[1] / b.ny);
    const double kz = (b.nz / 2) * (2.0 * M_PI * b.inv_h[2] / b.nz);
    return (int)std::floor(std::sqrt(kx * kx + ky * ky + kz * kz) + 0.5) + 1;
}

bool spectrum_supported(const BoxDesc &b) {
    const int n[3] = {b.nx, b.ny, b.nz};
    for (int d = 0; d < 3; ++d)
        if (n[d] > 2047) return false;
    // the shell histogram must fit in LDS, one block's partials and the per-shell second
    // moments in the rhs buffer (at least 20 bytes per point)
    const size_t hist = 2 * sizeof(double) * (size_t)spectrum_shells(b);
    return hist <= 64 * 1024 && hist + sizeof(double) * (size_t)spectrum_shells(b) <= 20 * b.n3;
}

static FftPlan fft_plan(int N, const double2 *tw) {
    FftPlan P{};
    P.N = N;
    P.nr = fft_factor(N, P.radix);
    P.ld = line_slots(N);
    P.dN = fastdiv((uint32_t)N);
    P.tw = tw;
    return P;
}

// LDS of the z pass: twiddles, lines, nh histograms (whose space takes one sum per wave at the end)
static size_t z_lds_bytes(int W, int N, int nshell, int nh) {
    return sizeof(double2) * ((size_t)tw_slots(N) + (size_t)W * line_slots(N)) + sizeof(double) * std::max(nh * (size_t)nshell, (size_t)8);
}

template <typename T, bool POW2, int NT>
static void spectrum_passes(const FftPlan &Px, const FftPlan &Py, const FftPlan &Pz, const SpecFields &F,
                            const SpecGeom &G, const T *u, double *part, unsigned nblocks, hipStream_t s) {
    constexpr int elems = NT * kFftPerThread;
    const int rows = F.ny * F.nz;
    // rows per block of the x pass: what the threads hold, fewer while that leaves less than
    // 512 blocks, but at least two elements per thread
    const int nl = std::max(1, std::min(elems / F.nx, std::max((rows + 511) / 512, 2 * NT / F.nx)));
    const unsigned gx = (unsigned)((rows + nl - 1) / nl);
    hipLaunchKernelGGL((k_fft_x<T, POW2, NT>), dim3(gx), dim3(NT), sizeof(double2) * ((size_t)nl * Px.ld + tw_slots(Px.N)), s, u,
                       G.n3, Px, F, nl);
    hipLaunchKernelGGL((k_fft_y<POW2, NT>), dim3((unsigned)((F.nrun[0] + F.nrun[1]) * F.nz)), dim3(NT),
                       sizeof(double2) * ((size_t)F.W * Py.ld + tw_slots(Py.N)), s, Py, F);
    const int ntask = (F.nrun[0] + F.nrun[1]) * F.ny;
    const size_t lds = z_lds_bytes(F.W, Pz.N, G.nshell, G.nh);
    hipLaunchKernelGGL((k_fft_z_bin<POW2, NT>), dim3(nblocks), dim3(NT), lds, s, Pz, F, G, ntask, part);
}

void launch_spectrum(const BoxDesc &b, int prec, hipStream_t s, const void *u, double *E, int nshell, double *mom) {
    const bool pow2 = !((b.nx & (b.nx - 1)) | (b.ny & (b.ny - 1)) | (b.nz & (b.nz - 1)));
    // Lengths are at least 8, so powers of two transform in registers; other lengths stage every
    // radix in LDS.  512 threads and 4096 elements per block in the large boxes of the former
    // (runs of 8 kx at 512^3 instead of 4, so that stores fill whole lines); else 256 and 2048
    const bool wide = pow2 && b.n3 >= (1u << 22) && std::max({b.nx, b.ny, b.nz}) <= 1024 &&
                      z_lds_bytes(4096 / b.nz, b.nz, nshell, 8) <= kSpecLdsMax;
    const int nt = wide ? 512 : 256, elems = nt * kFftPerThread;
    SpecFields F;
    F.nx = b.nx, F.ny = b.ny, F.nz = b.nz;
    F.W = kFftMaxW;
    while (F.W > 1 && F.W * std::max(b.ny, b.nz) > elems) F.W /= 2;
    F.nk[0] = b.nx, F.nk[1] = b.nx / 2 + 1;
    // a histogram for every wave while they fit beside lines of four kx, then fewer; the most
    // shells (4096) leave one wave's histogram and the longest line within the limit
    SpecGeom G;
    G.nh = nt / 64;
    while (z_lds_bytes(F.W, b.nz, nshell, G.nh) > kSpecLdsMax && (F.W > 1 || G.nh > 1))
        if (F.W > 4 || G.nh == 1) F.W /= 2;
        else G.nh /= 2;
    for (int f = 0; f < 2; ++f) F.nrun[f] = (F.nk[f] + F.W - 1) / F.W;
    // X1 takes 16 bytes per point, X2 at most 10, and the gaps of a large box (rows of 512
    // and more planes' lines) less than one; A and B hold 20 or 40, G 36 or 72
    const bool gaps = b.ny * (size_t)b.nz >= 16384 && b.nz >= 128;
    F.pz = gaps ? 3 : 0;
    F.sa = (size_t)F.W * ((size_t)b.ny * b.nz + (gaps ? 17 : 0));
    F.sb = (size_t)F.W * ((size_t)b.ny * (b.nz + F.pz) + (gaps ? 17 : 0));
    F.a[0] = (double2 *)b.A, F.a[1] = (double2 *)b.B;
    const size_t last = (size_t)F.nrun[0] - 1;  // the runs before the last are full
    F.b[0] = (double2 *)b.G;
    F.b[1] = F.b[0] + last * F.sb + (F.nk[0] - last * F.W) * (size_t)b.ny * (b.nz + F.pz);
    double2 *const tw = (double2 *)b.acc;
    hipLaunchKernelGGL(k_fft_twiddles, dim3(3), dim3(256), 0, s, tw, b.nx, b.ny, b.nz);
    const FftPlan Px = fft_plan(b.nx, tw), Py = fft_plan(b.ny, tw + b.nx), Pz = fft_plan(b.nz, tw + b.nx + b.ny);
    G.nx = b.nx, G.ny = b.ny, G.nz = b.nz, G.nshell = nshell, G.n3 = b.n3;
    G.kux = 2.0 * M_PI * b.inv_h[0] / b.nx;
    G.kuy = 2.0 * M_PI * b.inv_h[1] / b.ny;
    G.kuz = 2.0 * M_PI * b.inv_h[2] / b.nz;
    G.norm = 1.0 / ((double)b.n3 * (double)b.n3);
    // block partials, then the second moment, in the rhs buffer (at least 20 bytes per point)
    const size_t cap = (b.n3 * 20 - sizeof(double)) / (sizeof(double) * (size_t)(nshell + 1));
    const size_t ntask = (size_t)(F.nrun[0] + F.nrun[1]) * b.ny;
    const unsigned nb = (unsigned)std::max<size_t>(1, std::min<size_t>({cap, wide ? 512u : 1024u, ntask}));
    double *part = (double *)b.rhs;
    double *M2 = part + (size_t)nb * (nshell + 1);
    if (prec == CNS_FP64) {
        if (wide) spectrum_passes<double, true, 512>(Px, Py, Pz, F, G, (const double *)u, part, nb, s);
        else if (pow2) spectrum_passes<double, true, 256>(Px, Py, Pz, F, G, (const double *)u, part, nb, s);
        else spectrum_passes<double, false, 256>(Px, Py, Pz, F, G, (const double *)u, part, nb, s);
    } else {
        if (wide) spectrum_passes<float, true, 512>(Px, Py, Pz, F, G, (const float *)u, part, nb, s);
        else if (pow2) spectrum_passes<float, true, 256>(Px, Py, Pz, F, G, (const float *)u, part, nb, s);
        else spectrum_passes<float, false, 256>(Px, Py, Pz, F, G, (const float *)u, part, nb, s);
    }
    hipLaunchKernelGGL(k_spec_final, dim3((unsigned)nshell + 1), dim3(kPointThreads), 0, s, part, (int)nb, nshell, E, M2);
    hipLaunchKernelGGL(k_spec_mom, dim3(1), dim3(kPointThreads), 0, s, E, M2, nshell, mom);
}

}  // namespace cns
