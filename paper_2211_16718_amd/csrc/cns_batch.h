// cns_batch.h -- what the kernel files share: the walk over the virtual blocks of a batch,
// typed access to the boxes' arrays, the geometry of a sweep, launch arguments.
#pragma once
#include <hip/hip_runtime.h>

#include <type_traits>

#include "cns_internal.h"

namespace cns {

__device__ __forceinline__ int wrapi(int j, int n) { return j < 0 ? j + n : (j >= n ? j - n : j); }
// the same for any j >= -n (tile halos can reach several periods past a short line);
// the division only runs for lines shorter than the halo
__device__ __forceinline__ int wrapm(int j, int n) {
    int r = j < 0 ? j + n : j;
    r = r >= n ? r - n : r;
    return r >= n ? r % n : r;
}

// box owning virtual block vb: the last i with off[i] <= vb
__device__ __forceinline__ int find_box(const long long *off, int nbox, long long vb) {
    int lo = 0, hi = nbox;
    while (hi - lo > 1) {
        int mid = (lo + hi) >> 1;
        if (off[mid] <= vb) lo = mid;
        else hi = mid;
    }
    return lo;
}

// The virtual blocks a launched block runs.  Workgroups are dispatched to the 8 XCDs of
// the chip round-robin (block b on XCD b % 8), and each XCD has its own L2.  The
// virtual blocks are cut into one contiguous range per XCD, and the launched blocks of
// XCD x walk range x with a stride of their number, so blocks that touch neighbouring
// data (stencil halos) share an L2.  With one launched block per virtual block each
// runs exactly one; with fewer (a persistent launch, its grid sized to the blocks the
// chip holds at once) each loops over several.  Every virtual block runs exactly once
// for any grid size.
struct VbRange {
    long long vb, end, stride;
};
__device__ __forceinline__ VbRange vb_range(long long total) {
    const long long G = gridDim.x, b = blockIdx.x;
    const long long X = G < 8 ? G : 8;  // ranges: one per XCD that has blocks
    const long long x = b % X, l = b / X;
    const long long nbx = G / X + (x < G % X ? 1 : 0);
    const long long q = total / X, r = total % X;
    const long long lo = x * q + (x < r ? x : r), hi = lo + q + (x < r ? 1 : 0);
    return VbRange{lo + l, hi, nbx};
}

// the launch with the per-call record of a graph replay applied (read once per kernel)
__device__ __forceinline__ Launch with_params(Launch L) {
    if (L.gp) {
        L.u_ov = L.gp->u;
        L.dt_ov = L.gp->dt;
        L.diag = L.gp->diag;
    }
    return L;
}

// Pointers into HBM taken from the device tables are generic (flat) pointers to the
// compiler, and accesses through them become FLAT instructions, which count against
// the LDS counter as well as the vector-memory counter: every wait for an LDS read then
// also waits for all HBM loads in flight, which undoes the loads issued ahead of the
// arithmetic.  The kernels cast them to the global address space (HBM), whose
// accesses count against the vector-memory counter only.
template <typename T>
using gptr = __attribute__((address_space(1))) T *;
template <typename T>
__device__ __forceinline__ gptr<T> glob(T *p) {
    return (gptr<T>)p;
}

// A value all lanes hold alike (read from the box table) moved into scalar registers.
// The compiler cannot prove that table reads are the same on every lane; marked
// uniform, the pointers stay in scalar registers across the loops instead of being
// copied back from vector registers before each access.
__device__ __forceinline__ uint64_t uni64(uint64_t v) {
    const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)v);
    const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)(v >> 32));
    return ((uint64_t)hi << 32) | lo;
}
template <typename T>
__device__ __forceinline__ gptr<T> uni(gptr<T> p) {
    return (gptr<T>)uni64((uint64_t)p);
}

// Component c of a component-major array (component c at element c * n3) at a lane's
// byte offset: the array base and the component offset are uniform and stay in scalar
// registers, and every load and store of a point shares the lane's one 32-bit offset
// register (global memory instructions with a scalar base address).  Needs
// n3 * 8 < 2^32, which plan and ensemble creation check.
template <typename T>
__device__ __forceinline__ gptr<T> elem(gptr<T> a, size_t n3, int c, uint32_t boff) {
    using Byte = typename std::conditional<std::is_const<T>::value, const char, char>::type;
    return (gptr<T>)((gptr<Byte>)(a + (size_t)c * n3) + boff);
}

__device__ __forceinline__ const void *state_ptr(const BoxDesc &b, const Launch &L, int which) {
    if (which == BUF_U) return L.u_ov ? L.u_ov : b.u;
    if (which == BUF_A) return L.a_ov ? L.a_ov : b.A;
    return L.b_ov ? L.b_ov : b.B;
}

// The halo ring of a kViscTX x kViscTY tile in its (kViscTX + 4) x (kViscTY + 4) staging
// plane: rows 0, 1, kViscTY + 2, kViscTY + 3 in full, then columns 0, 1, kViscTX + 2,
// kViscTX + 3 of the rows between.  Thread t < kViscRing owns ring position t.
constexpr int kViscRingRows = 4 * (kViscTX + 4);
constexpr int kViscRing = kViscRingRows + 4 * kViscTY;
static_assert(kViscRing <= kDiagThreads, "one halo point per thread");
__device__ __forceinline__ void ring_pos(int t, int &hx, int &hy) {
    if (t < kViscRingRows) {
        const int r = t / (kViscTX + 4);
        hx = t % (kViscTX + 4);
        hy = r < 2 ? r : kViscTY + r;
    } else {
        const int q = t - kViscRingRows, c = q & 3;
        hy = 2 + (q >> 2);
        hx = c < 2 ? c : kViscTX + c;
    }
}

// geometry of a sweep along DIR: lanes run over the plane normal to DIR (p fastest)
struct SweepGeom {
    int nline, np, npq;
    size_t lstride, pstride, qstride;
};
template <int DIR>
__host__ __device__ __forceinline__ SweepGeom sweep_geom(int nx, int ny, int nz) {
    const size_t sy = (size_t)nx, sz = (size_t)nx * ny;
    if (DIR == 0) return SweepGeom{nx, ny, ny * nz, 1, sy, sz};
    if (DIR == 1) return SweepGeom{ny, nx, nx * nz, sy, 1, sz};
    return SweepGeom{nz, nx, nx * ny, sz, 1, sy};
}

// ----------------------------------------------------------------------------
// host side
// ----------------------------------------------------------------------------
inline long long cdiv(long long a, long long b) { return (a + b - 1) / b; }

inline Launch make_launch(const Batch &bt, int fam) {
    Launch L{};
    L.gp = bt.gp;
    L.boxes = bt.d_boxes;
    L.off = bt.d_off[fam];
    L.nbox = bt.nbox;
    L.total = bt.total[fam];
    return L;
}

inline Launch with_family(const Batch &bt, Launch L, int fam) {
    L.off = bt.d_off[fam];
    L.total = bt.total[fam];
    return L;
}

inline unsigned grid_for(long long total) {
    const long long cap = 1ll << 30;
    return (unsigned)(total < cap ? total : cap);
}

// launched blocks of family fam: bt.grid[fam] when set (a persistent launch), else one
// per virtual block
inline unsigned grid_of(const Batch &bt, int fam, long long total) {
    const long long g = bt.grid[fam];
    return grid_for(g > 0 && g < total ? g : total);
}

}  // namespace cns
