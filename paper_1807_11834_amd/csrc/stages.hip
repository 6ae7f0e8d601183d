// stages.hip -- restriction, particle sampling, drag, prolongation and the FP64
// conservation sums of one coupling step (deposition is in deposit.hip).
//
// Kernel order on the caller's stream (after binning/sorting, sort.hip):
//
//   deposit phi    (deposit.hip), which also makes the sorted copy sp = (x, y,
//                  z, d) of the particles from the packed input-order copy that
//                  binning wrote (clamped into the box).
//   k_restrict     one thread per bulk cell streams its r^3 fine children of
//                  u, v, w, p (one 16-byte row load per (z, y) child row for
//                  r = 4) and writes the compensated averages U, P.
//   k_restrict_brick  the same restriction tiled in 8x4x2-cell bricks with the
//                  fine-grid lookup fused: the brick's fine u, v, w stay in LDS
//                  and its particles are sampled from there (fine trilinear
//                  velocity, void fraction from a haloed copy of phi), so the
//                  fine lookup costs no extra pass over the fine grid.
//   k_sample       the same sampling for the bulk and given velocity sources.
//   k_restrict_alpha  two-fluid drag: bulk liquid fraction, average of the fine
//                  children; k_pack_alpha8 then stores each cell's 2x2x2
//                  stencil corners as one record for the drag's lookups.
//   k_drag         drag and explicit Euler advection in input order (coalesced);
//                  with the semi-implicit split also (beta, beta u_p).
//   deposit force  (deposit.hip), with the bulk pressure gradient; then the
//                  semi-implicit K, KU when requested.
//   k_prolong      a tile of 256 bulk cells per work item, one launch for eps,
//                  F_fpi (and K, KU): conservative trilinear
//                  T_f + D_c from the tile staged in LDS.
//   k_diag         fixed-order reduction of the per-workgroup FP64 partials.
#include <algorithm>
#include <type_traits>

#include "common.hpp"
#include "launch.hpp"
#include "sample.hpp"

namespace cpl {

// ---------------------------------------------------------------------------
// Row loads of R consecutive fine values (16-byte vector loads where possible)
// ---------------------------------------------------------------------------
template <typename T, int R> struct Row { T v[R]; };

template <typename T, int N> using NtVec = T __attribute__((ext_vector_type(N)));

// STREAM: non-temporal loads, for fine rows that no later kernel of the step
// reads again (k_restrict, k_restrict_alpha); the brick kernel's rows use
// ordinary loads, since the stencils of its particles near a brick face read
// the neighbouring bricks' rows from the cache.
template <typename T, int N, bool STREAM> __device__ __forceinline__ NtVec<T, N> load_vec(const T *__restrict__ p) {
    const NtVec<T, N> *q = reinterpret_cast<const NtVec<T, N> *>(p);
    if constexpr (STREAM) return __builtin_nontemporal_load(q);
    else return *q;
}

template <typename T, int R, bool STREAM = false>
__device__ __forceinline__ Row<T, R> load_row(const T *__restrict__ p) {
    Row<T, R> r;
    if constexpr (std::is_same<T, float>::value && R == 4) {
        const NtVec<float, 4> q = load_vec<float, 4, STREAM>(p);
        r.v[0] = q.x; r.v[1] = q.y; r.v[2] = q.z; r.v[3] = q.w;
    } else if constexpr (std::is_same<T, float>::value && R == 2) {
        const NtVec<float, 2> q = load_vec<float, 2, STREAM>(p);
        r.v[0] = q.x; r.v[1] = q.y;
    } else if constexpr (std::is_same<T, double>::value && R == 4) {
        const NtVec<double, 2> a = load_vec<double, 2, STREAM>(p), b = load_vec<double, 2, STREAM>(p + 2);
        r.v[0] = a.x; r.v[1] = a.y; r.v[2] = b.x; r.v[3] = b.y;
    } else if constexpr (std::is_same<T, double>::value && R == 2) {
        const NtVec<double, 2> a = load_vec<double, 2, STREAM>(p);
        r.v[0] = a.x; r.v[1] = a.y;
    } else {
        for (int k = 0; k < R; ++k) r.v[k] = p[k];
    }
    return r;
}

// Fine-grid rows written once and not read again in the step: non-temporal
// stores, so that the 4 GB written per prolongation do not sit dirty in the
// caches and slow the next kernels while they are written back.
template <typename T, int R> __device__ __forceinline__ void store_row(T *__restrict__ p, const T *v) {
    if constexpr (std::is_same<T, float>::value && R == 4) {
        const NtVec<float, 4> q = {v[0], v[1], v[2], v[3]};
        __builtin_nontemporal_store(q, reinterpret_cast<NtVec<float, 4> *>(p));
    } else if constexpr (std::is_same<T, float>::value && R == 2) {
        const NtVec<float, 2> q = {v[0], v[1]};
        __builtin_nontemporal_store(q, reinterpret_cast<NtVec<float, 2> *>(p));
    } else if constexpr (std::is_same<T, double>::value && R == 4) {
        const NtVec<double, 2> q0 = {v[0], v[1]}, q1 = {v[2], v[3]};
        __builtin_nontemporal_store(q0, reinterpret_cast<NtVec<double, 2> *>(p));
        __builtin_nontemporal_store(q1, reinterpret_cast<NtVec<double, 2> *>(p) + 1);
    } else if constexpr (std::is_same<T, double>::value && R == 2) {
        const NtVec<double, 2> q = {v[0], v[1]};
        __builtin_nontemporal_store(q, reinterpret_cast<NtVec<double, 2> *>(p));
    } else {
        for (int k = 0; k < R; ++k) __builtin_nontemporal_store(v[k], p + k);
    }
}

// ---------------------------------------------------------------------------
// Particle stage: void fraction and fluid velocity at the particle, drag
// (Eq. DragLaw with the Di Felice voidage function), optional Euler advection.
// ---------------------------------------------------------------------------
// Per particle in the sorted order: sample_one() with the handle's velocity
// source, written to uf4[id] = (u, v, w, eps_p) for the input-order drag kernel.
// KB particles per thread are sampled together so that all their gathers are in
// flight at once.
template <typename T, int KB>
__device__ __forceinline__ void sample_particles(const int64_t (&idx)[KB], const StepArgs<T> &a) {
    const vec4<T> *__restrict__ sp = a.sp;
    const int32_t *__restrict__ perm = a.perm;
    vec4<T> q[KB];
    int64_t p[KB];
#pragma unroll
    for (int k = 0; k < KB; ++k) {
        const int64_t i = idx[k] >= 0 ? idx[k] : 0;
        q[k] = sp[i];
        p[k] = perm[i];
        if (p[k] < 0 || p[k] >= a.n) p[k] = 0;   // perm is a permutation of [0, n)
    }
    vec4<T> s[KB];
#pragma unroll
    for (int k = 0; k < KB; ++k) s[k] = sample_one(q[k], a, a.vel_source);
#pragma unroll
    for (int k = 0; k < KB; ++k)
        if (idx[k] >= 0) a.uf4[p[k]] = s[k];
}

// ---------------------------------------------------------------------------
// Restriction fine -> bulk
// ---------------------------------------------------------------------------
// Sums of the r^3 fine children, per fine child plane and then the planes in
// order, under the step's sum mode.  Kahan (FP32): each plane is a Kahan sum and
// the planes are combined as s_0, -c_0, s_1, -c_1, ... in a Kahan sum; the
// average's residue lo = -c / r^3 carries the rest of the pressure for the
// gradient.  Wide (FP32 storage): the children are widened to FP64 and summed
// there; with at most 64 terms the sum is within 64 FP64 roundings of exact, so
// its FP32 rounding is the correctly rounded average in all but rare ties, and
// the FP32 residue lo = S - hi carries the rest of the pressure; one convert and
// one FP64 add per child instead of Kahan's four instructions.  Plain: the FP64
// mode and naive FP32 sum in their own type.
template <typename T, int SM> struct ChildSum {
    static constexpr bool kWide = std::is_same<T, float>::value && SM == kSumWide;
    using W = typename std::conditional<kWide, double, T>::type;
    static constexpr bool kComp = SM == kSumKahan;   // Kahan in T
    Acc<W, kComp> acc;
    __device__ __forceinline__ void add(T v) { acc.add(W(v)); }
    // a plane's sum (s, with its compensation c) added to the cell's
    __device__ __forceinline__ void add_plane(W ps, W pc) {
        acc.add(ps);
        if constexpr (kComp) acc.add(-pc);
    }
    // the average, and what its rounding leaves out (the scale 1/r^3 is a power
    // of two, so the scaling is exact)
    __device__ __forceinline__ T hi(T inv) const { return T(acc.s * W(inv)); }
    __device__ __forceinline__ T lo(T inv) const {
        if constexpr (kWide) return T(acc.s * W(inv) - W(hi(inv)));
        else return -acc.c * inv;
    }
};

// Fields F0 .. F1 - 1 of (u, v, w, p): all four for the bulk, given and learned
// velocity sources, the pressure alone beside the brick kernel (which restricts
// u, v, w).
template <typename T, int R, int SM, int F0, int F1>
__global__ __launch_bounds__(kBlock) void k_restrict(StepArgs<T> a) {
    const Geo<T> &g = a.g;
    const int64_t tile = xcd_tile(blockIdx.x, gridDim.x);
    const int64_t c = tile * kBlock + threadIdx.x;
    if (c < g.ncell) {
        int cx, cy, cz;
        decode_cell(c, g.nb, cx, cy, cz);
        const int64_t nfx = g.nf[0], nfxy = (int64_t)g.nf[0] * g.nf[1];
        const int64_t base = (int64_t)R * cz * nfxy + (int64_t)R * cy * nfx + (int64_t)R * cx;
        const T inv = T(1) / T(R * R * R);
#pragma unroll
        for (int f = F0; f < F1; ++f) {
            const T *__restrict__ q = a.fine[f] + base;
            Row<T, R> rows[R][R];
#pragma unroll
            for (int lz = 0; lz < R; ++lz)
#pragma unroll
                for (int ly = 0; ly < R; ++ly) rows[lz][ly] = load_row<T, R, true>(q + lz * nfxy + ly * nfx);
            // per fine child plane, then the planes in order (with a Kahan sum,
            // s_0, -c_0, s_1, ...): the same sums as the brick-tiled kernel
            ChildSum<T, SM> acc;
#pragma unroll
            for (int lz = 0; lz < R; ++lz) {
                ChildSum<T, SM> plane;
#pragma unroll
                for (int ly = 0; ly < R; ++ly)
#pragma unroll
                    for (int lx = 0; lx < R; ++lx) plane.add(rows[lz][ly].v[lx]);
                acc.add_plane(plane.acc.s, plane.acc.c);
            }
            const T val = acc.hi(inv);
            if (f < 3) {
                a.U[f * g.ncell + c] = val;
            } else {
                a.P[c] = val;
                // keep the rest of the average so that the pressure gradient can
                // difference (hi + lo) instead of the rounded hi
                a.Plo[c] = acc.lo(inv);
            }
        }
    }
}

// The same restrictions for r = 4 with four threads per bulk cell, one per fine
// child plane (64 cells per workgroup): a thread loads its plane's 4 x 4 child
// values of every field with streaming loads and sums them, and the cell's four
// plane sums are combined in order through cross-lane reads, the sums of the
// per-cell kernel above bit for bit.  A wave's row load covers 16 cells x 4
// planes, whole 128-byte lines, and each thread keeps a quarter of the per-cell
// kernel's loads in flight.  ALPHA: the liquid fraction instead of (u, v, w, p).
constexpr int kPlaneCells = kBlock / 4;   // bulk cells per workgroup

template <typename T, int SM, int F0, int F1, bool ALPHA>
__global__ __launch_bounds__(kBlock) void k_restrict_planes(StepArgs<T> a) {
    constexpr int R = 4, NF = ALPHA ? 1 : F1 - F0;
    const Geo<T> &g = a.g;
    const int t = (int)threadIdx.x, lane = t % kWave, rz = t & 3;
    const int64_t c = xcd_tile(blockIdx.x, gridDim.x) * kPlaneCells + (t >> 2);
    const bool inside = c < g.ncell;
    int cx, cy, cz;
    decode_cell(inside ? c : g.ncell - 1, g.nb, cx, cy, cz);   // every lane takes part in the cross-lane reads
    const int64_t nfx = g.nf[0], nfxy = (int64_t)g.nf[0] * g.nf[1];
    const int64_t base = ((int64_t)R * cz + rz) * nfxy + (int64_t)R * cy * nfx + (int64_t)R * cx;
    Row<T, R> rows[NF][R];
#pragma unroll
    for (int f = 0; f < NF; ++f) {
        const T *__restrict__ q = (ALPHA ? a.fine_alpha : a.fine[F0 + f]) + base;
#pragma unroll
        for (int ry = 0; ry < R; ++ry) rows[f][ry] = load_row<T, R, true>(q + ry * nfx);
    }
    const T inv = T(1) / T(R * R * R);
    const int l0 = lane & ~3;
#pragma unroll
    for (int f = 0; f < NF; ++f) {
        ChildSum<T, SM> plane;
#pragma unroll
        for (int ry = 0; ry < R; ++ry)
#pragma unroll
            for (int rx = 0; rx < R; ++rx) plane.add(rows[f][ry].v[rx]);
        ChildSum<T, SM> acc;
#pragma unroll
        for (int k = 0; k < R; ++k) {
            const auto sk = __shfl(plane.acc.s, l0 + k, kWave);
            const auto ck = ChildSum<T, SM>::kComp ? __shfl(plane.acc.c, l0 + k, kWave) : plane.acc.c;
            acc.add_plane(sk, ck);
        }
        if (inside && rz == 0) {
            if constexpr (ALPHA) {
                a.alpha[c] = acc.hi(inv);
            } else if (F0 + f < 3) {
                a.U[(F0 + f) * g.ncell + c] = acc.hi(inv);
            } else {
                a.P[c] = acc.hi(inv);
                a.Plo[c] = acc.lo(inv);
            }
        }
    }
}

// Restriction of the liquid volume fraction (two-fluid drag): the bulk alpha is
// the average of the r^3 fine children (the volume average that defines alpha),
// summed per fine child plane and then the planes in order, as for U and P.
template <typename T, int R, int SM>
__global__ __launch_bounds__(kBlock) void k_restrict_alpha(StepArgs<T> a) {
    const Geo<T> &g = a.g;
    const int64_t tile = xcd_tile(blockIdx.x, gridDim.x);
    const int64_t c = tile * kBlock + threadIdx.x;
    if (c >= g.ncell) return;
    int cx, cy, cz;
    decode_cell(c, g.nb, cx, cy, cz);
    const int64_t nfx = g.nf[0], nfxy = (int64_t)g.nf[0] * g.nf[1];
    const T *__restrict__ q = a.fine_alpha + (int64_t)R * cz * nfxy + (int64_t)R * cy * nfx + (int64_t)R * cx;
    Row<T, R> rows[R][R];
#pragma unroll
    for (int lz = 0; lz < R; ++lz)
#pragma unroll
        for (int ly = 0; ly < R; ++ly) rows[lz][ly] = load_row<T, R, true>(q + lz * nfxy + ly * nfx);
    ChildSum<T, SM> acc;
#pragma unroll
    for (int lz = 0; lz < R; ++lz) {
        ChildSum<T, SM> plane;
#pragma unroll
        for (int ly = 0; ly < R; ++ly)
#pragma unroll
            for (int lx = 0; lx < R; ++lx) plane.add(rows[lz][ly].v[lx]);
        acc.add_plane(plane.acc.s, plane.acc.c);
    }
    a.alpha[c] = acc.hi(T(1) / T(R * R * R));
}

// The bulk alpha at the eight cells cell + {0,1}^3 (clamped into the grid), as
// one 8-value record per cell: the drag kernel runs in input order, and a
// particle's trilinear stencil (whose lower corner is the record's cell) is
// then one 32-byte read instead of reads from four rows of the bulk grid.
template <typename T>
__global__ __launch_bounds__(kBlock) void k_pack_alpha8(StepArgs<T> a) {
    const Geo<T> &g = a.g;
    const int64_t c = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (c >= g.ncell) return;
    int cx, cy, cz;
    decode_cell(c, g.nb, cx, cy, cz);
    const int64_t nx = g.nb[0], nxy = nx * g.nb[1];
    const int64_t xs[2] = {cx, cx + 1 < g.nb[0] ? cx + 1 : cx};
    const int64_t ys[2] = {cy * nx, (cy + 1 < g.nb[1] ? cy + 1 : cy) * nx};
    const int64_t zs[2] = {cz * nxy, (cz + 1 < g.nb[2] ? cz + 1 : cz) * nxy};
    vec4<T> r[2];
    for (int dz = 0; dz < 2; ++dz) {
        r[dz].x = a.alpha[zs[dz] + ys[0] + xs[0]];
        r[dz].y = a.alpha[zs[dz] + ys[0] + xs[1]];
        r[dz].z = a.alpha[zs[dz] + ys[1] + xs[0]];
        r[dz].w = a.alpha[zs[dz] + ys[1] + xs[1]];
    }
    vec4<T> *out = reinterpret_cast<vec4<T> *>(a.alpha8) + 2 * c;
    out[0] = r[0];
    out[1] = r[1];
}

// Trilinear alpha at a particle from its stencil record, in the arithmetic
// order of trilin() (the same value bit for bit).
template <typename T>
__device__ __forceinline__ T trilin_alpha8(const T *__restrict__ alpha8, const Axis<T> &ax, const Axis<T> &ay,
                                           const Axis<T> &az, const int nb[3]) {
    const vec4<T> *r = reinterpret_cast<const vec4<T> *>(alpha8) +
                       2 * (((int64_t)az.lo * nb[1] + ay.lo) * nb[0] + ax.lo);
    const vec4<T> lo = r[0];
    const vec4<T> hi = az.hi != az.lo ? r[1] : lo;
    const bool ox = ax.hi != ax.lo, oy = ay.hi != ay.lo;
    // corner [z][y][x] of the stencil: x, y offsets 0 at a folded wall
    const T z0y0x0 = lo.x, z0y0x1 = ox ? lo.y : lo.x, z0y1x0 = oy ? lo.z : lo.x,
            z0y1x1 = oy ? (ox ? lo.w : lo.z) : (ox ? lo.y : lo.x);
    const T z1y0x0 = hi.x, z1y0x1 = ox ? hi.y : hi.x, z1y1x0 = oy ? hi.z : hi.x,
            z1y1x1 = oy ? (ox ? hi.w : hi.z) : (ox ? hi.y : hi.x);
    const T sx = T(1) - ax.t, sy = T(1) - ay.t, sz = T(1) - az.t;
    const T c00 = sx * z0y0x0 + ax.t * z0y0x1;
    const T c01 = sx * z0y1x0 + ax.t * z0y1x1;
    const T c10 = sx * z1y0x0 + ax.t * z1y0x1;
    const T c11 = sx * z1y1x0 + ax.t * z1y1x1;
    const T c0 = sy * c00 + ay.t * c01;
    const T c1 = sy * c10 + ay.t * c11;
    return sz * c0 + az.t * c1;
}

// Restriction of the velocity with the fine-grid lookup, tiled in bricks of
// 8 x 4 x 2 bulk cells.  Filling a brick: four threads per cell (one per fine
// child plane z) for u and v and four for w, each loads its plane's r x r rows of
// a component, stores them in LDS and sums its plane (compensated); the four
// plane sums are combined in order through cross-lane reads (the pressure is
// restricted by k_restrict before this kernel).  The brick's particles (8 rows of
// up to 8 cells, contiguous in the sorted order, flattened over the threads) then
// take their trilinear fine velocity from LDS when all eight fine nodes lie in
// the brick (from global memory when the stencil crosses a brick face) and their
// void fraction from a haloed copy of phi in LDS.  The brick is 8r fine cells wide
// along x (one 128-byte line per row for r = 4 in FP32).
// One workgroup per brick: fill, then the particles.  In a packed bed of 512 x 512
// x 1024 fine cells and 10 million particles the fill alone takes 620 of the 1000
// us (3.2 GB), the scattered stores of the results 200 and the particles at brick
// faces 90.  Lanes along x in the fill (rather than four planes of a cell next to
// each other, whose LDS stores conflict): 1042 -> 1016; 512 threads instead of
// 256, so that a brick's particles (a few hundred) are one batch of one particle
// per thread: -> 1001, and 95 -> 90 for 256^3 cells with 2 million.  (Loading the
// first particles before the barrier: 1039; bricks ordered in columns of two to
// eight along z, or dealt to the XCDs in rows or layers: no faster.)
constexpr int kBrickX = 8, kBrickY = 4, kBrickZ = 2;
constexpr int kBrickFill = 4 * kBrickX * kBrickY * kBrickZ;   // threads that fill one component
// HALVES = 2: the first half of 512 threads fills u and v, the other w, phi and the
// particle rows; 1: each of 256 fills all three.  Ratio 4 takes 512, and so do fewer
// bricks than fill the chip (two per compute unit), whose particles are then one
// batch (17 x 13 x 19 cells of ratio 2 with 20,000 particles, 7.6 us; with 256
// threads 9.0).  More bricks of a smaller ratio have little to fill, half of the
// threads or more idle meanwhile: 128 x 128 x 256 cells of ratio 1 with 100,000
// particles, 115 us with 256 threads and 200 with 512, in FP64 163 and 367; 100^3 of
// ratio 2 with 50,000, 36 and 57.
template <int HALVES> constexpr int kBrickThreads = HALVES * kBrickFill;
constexpr int64_t kBrickFew = 512;
// Waves per SIMD asked of the compiler: FP64 would take 98 registers, four waves; in
// 96, five (the FP64 figure above: 189 -> 163 us; six spill, 174).
template <typename T, int HALVES> struct BrickWaves {
    static constexpr int value = HALVES == 1 && sizeof(T) == 8 ? 5 : 1;
};
constexpr int kBrickRows = kBrickY * kBrickZ;                                     // particle rows of a brick
constexpr int kBrickHalo = (kBrickX + 2) * (kBrickY + 2) * (kBrickZ + 2);         // phi with a one-cell halo

template <typename T, int R> struct BrickLds {
    T sv[3][kBrickZ * R][kBrickY * R][kBrickX * R];
    T sphi[kBrickZ + 2][kBrickY + 2][kBrickX + 2];
    int32_t cnt[kBrickRows];   // particles of each row
    int32_t beg[kBrickRows];   // first sorted position of each row
};

template <typename T> struct BrickGrid {
    int bnx, bny;
    __device__ __forceinline__ void origin(int64_t brick, int &ox, int &oy, int &oz) const {
        const uint32_t row = (uint32_t)brick / (uint32_t)bnx, layer = row / (uint32_t)bny;   // fewer than 2^31 bricks
        ox = (int)((uint32_t)brick - row * (uint32_t)bnx) * kBrickX;
        oy = (int)(row - layer * (uint32_t)bny) * kBrickY;
        oz = (int)layer * kBrickZ;
    }
};

// Fill the brick at (ox, oy, oz) into L and (if write_u) write its U; thread t of
// kBrickThreads<HALVES>.
template <typename T, int R, int SM, int HALVES>
__device__ __forceinline__ void brick_fill(const StepArgs<T> &a, BrickLds<T, R> &L, int t, int ox, int oy, int oz,
                                           bool write_u) {
    constexpr int HX = kBrickX + 2, HY = kBrickY + 2;
    const Geo<T> &g = a.g;
    const int lane = t % kWave;
    constexpr bool kSplit = HALVES == 2;
    const bool upper = kSplit && t >= kBrickFill;   // a wave is in one half
    const bool rest = upper || !kSplit;             // phi and the particle rows
    t %= kBrickFill;
    // components of this thread: f0, f0 + 1, ... (nf of them)
    constexpr int NF = kSplit ? 2 : 3;
    const int f0 = upper ? 2 : 0, nf = upper ? 1 : NF;
    // cell of the brick and fine child plane: the eight lanes along x read and
    // write a contiguous row
    const int lx = t % kBrickX, rz = (t / kBrickX) % 4, ly = (t / (4 * kBrickX)) % kBrickY, lz = t / (4 * kBrickX * kBrickY);
    const int cx = ox + lx, cy = oy + ly, cz = oz + lz;
    const bool inside = cx < g.nb[0] && cy < g.nb[1] && cz < g.nb[2];
    const int64_t nx = g.nb[0], nxy = (int64_t)g.nb[0] * g.nb[1];
    const int64_t nfx = g.nf[0], nfxy = (int64_t)g.nf[0] * g.nf[1];
    // Every load of the fill is issued before the first LDS write: the brick's
    // particle rows (their first sorted position and count), phi with its halo
    // (indices clamped at the walls) and the fine rows, so that a workgroup
    // waits for one memory round trip instead of three.
    static_assert(kBrickHalo <= kBrickFill, "one halo value per thread");
    int32_t seg0 = 0, seg1 = 0;
    if (rest && t < kBrickRows) {
        const int wx = (ox + kBrickX < g.nb[0]) ? kBrickX : g.nb[0] - ox;
        const int ry = oy + t % kBrickY, rzz = oz + t / kBrickY;
        if (ry < g.nb[1] && rzz < g.nb[2]) {
            const int64_t c0 = ox + nx * ry + nxy * rzz;
            seg0 = a.start[c0];
            seg1 = a.start[c0 + wx];
        }
    }
    const int hx = t % HX, hy = (t / HX) % HY, hz = t / (HX * HY);
    T ph = T(0);
    if (rest && t < kBrickHalo) {
        const int gx = clampi(ox - 1 + hx, g.nb[0]), gy = clampi(oy - 1 + hy, g.nb[1]), gz = clampi(oz - 1 + hz, g.nb[2]);
        ph = a.phi[gx + nx * gy + nxy * gz];
    }
    const bool work = inside && rz < R;
    const int64_t base = ((int64_t)R * cz + rz) * nfxy + (int64_t)R * cy * nfx + (int64_t)R * cx;
    const T inv = T(1) / T(R * R * R);
    Row<T, R> rows[NF][R];
#pragma unroll
    for (int i = 0; i < NF; ++i) {
        if (i >= nf) break;
        const T *__restrict__ q = (upper ? a.fine[2] : a.fine[i]) + base;
        if (work) {
#pragma unroll
            for (int ry = 0; ry < R; ++ry) rows[i][ry] = load_row<T, R>(q + ry * nfx);
        }
    }
    if (rest && t < kBrickRows) {
        const int32_t b0 = seg_clamp(seg0, a.n);
        L.beg[t] = b0;
        L.cnt[t] = seg_clamp(seg1, a.n) - b0;
    }
    if (rest && t < kBrickHalo) L.sphi[hz][hy][hx] = ph;
#pragma unroll
    for (int i = 0; i < NF; ++i) {
        if (i >= nf) break;
        const int f = f0 + i;
        ChildSum<T, SM> plane;
        if (work) {
#pragma unroll
            for (int ry = 0; ry < R; ++ry)
#pragma unroll
                for (int rx = 0; rx < R; ++rx) plane.add(rows[i][ry].v[rx]);
#pragma unroll
            for (int ry = 0; ry < R; ++ry)
#pragma unroll
                for (int rx = 0; rx < R; ++rx) L.sv[f][lz * R + rz][ly * R + ry][lx * R + rx] = rows[i][ry].v[rx];
        }
        // the planes of this cell in order (with a Kahan sum, s_0, -c_0, s_1,
        // ...), read from the cell's four lanes; the plane-0 lane writes the
        // average
        ChildSum<T, SM> acc;
        const int l0 = lane - kBrickX * rz;
#pragma unroll
        for (int k = 0; k < R; ++k) {
            const auto sk = __shfl(plane.acc.s, l0 + kBrickX * k, kWave);
            const auto ck = ChildSum<T, SM>::kComp ? __shfl(plane.acc.c, l0 + kBrickX * k, kWave) : plane.acc.c;
            acc.add_plane(sk, ck);
        }
        if (write_u && inside && rz == 0) a.U[f * g.ncell + (cx + nx * cy + nxy * cz)] = acc.hi(inv);
    }
}

// The particles of the filled brick at (ox, oy, oz): thread t of nt, batches
// first, first + step, ... of one particle per thread.
template <typename T, int R>
__device__ __forceinline__ void brick_particles(const StepArgs<T> &a, const BrickLds<T, R> &L, int t, int nt, int first,
                                                int step, int ox, int oy, int oz) {
    constexpr int FX = kBrickX * R, FY = kBrickY * R, FZ = kBrickZ * R;
    const Geo<T> &g = a.g;
    int32_t pre[kBrickRows + 1];   // particles before each row
    pre[0] = 0;
#pragma unroll
    for (int r = 0; r < kBrickRows; ++r) pre[r + 1] = pre[r] + L.cnt[r];
    const int total = pre[kBrickRows];
    const int fx0 = ox * R, fy0 = oy * R, fz0 = oz * R;
    for (int j = t + first * nt; j < total; j += step * nt) {
        int r = 0;
#pragma unroll
        for (int q = 1; q < kBrickRows; ++q) r += (pre[q] <= j) ? 1 : 0;
        const int64_t i = L.beg[r] + (j - pre[r]);
        const vec4<T> q = a.sp[i];
        int64_t p = a.perm[i];
        if (p < 0 || p >= a.n) p = 0;   // perm is a permutation of [0, n)
        vec4<T> s;
        // fine trilinear velocity: from LDS when the eight nodes lie in the brick
        const Axis<T> ax = cic_axis(q.x, g.sf[0], g.nf[0]);
        const Axis<T> ay = cic_axis(q.y, g.sf[1], g.nf[1]);
        const Axis<T> az = cic_axis(q.z, g.sf[2], g.nf[2]);
        const int xl = ax.lo - fx0, xh = ax.hi - fx0, yl = ay.lo - fy0, yh = ay.hi - fy0, zl = az.lo - fz0,
                  zh = az.hi - fz0;
        if (xl >= 0 && xh < FX && yl >= 0 && yh < FY && zl >= 0 && zh < FZ) {
            const T tx = ax.t, ty = ay.t, tz = az.t, sx = T(1) - tx, sy = T(1) - ty, sz = T(1) - tz;
            T u[3];
#pragma unroll
            for (int f = 0; f < 3; ++f) {
                // rounded as written, in this lookup's own order (see trilin_rows)
                auto row = [&](int z, int y) { return dfma(sx, L.sv[f][z][y][xl], tx * L.sv[f][z][y][xh]); };
                const T e0 = dfma(sy, row(zl, yl), ty * row(zl, yh));
                const T e1 = dfma(sy, row(zh, yl), ty * row(zh, yh));
                u[f] = f < 2 ? dfma(sz, e0, tz * e1) : dfma(tz, e1, sz * e0);
            }
            s.x = u[0];
            s.y = u[1];
            s.z = u[2];
        } else {
            fine_velocity(q, a, s.x, s.y, s.z);
        }
        // void fraction at the particle from the haloed phi (its stencil is the
        // containing cell and a neighbour, always inside the halo)
        if (a.cic) {
            // (x rounded as this lookup always has: see node_units_rounded)
            const Axis<T> bx = cic_axis_at(node_units_rounded(q.x, g.sb[0]), g.nb[0]);
            const Axis<T> by = cic_axis(q.y, g.sb[1], g.nb[1]);
            const Axis<T> bz = cic_axis(q.z, g.sb[2], g.nb[2]);
            const int hxl = bx.lo - ox + 1, hxh = bx.hi - ox + 1, hyl = by.lo - oy + 1, hyh = by.hi - oy + 1,
                      hzl = bz.lo - oz + 1, hzh = bz.hi - oz + 1;
            const T f000 = L.sphi[hzl][hyl][hxl], f001 = L.sphi[hzl][hyl][hxh], f010 = L.sphi[hzl][hyh][hxl],
                    f011 = L.sphi[hzl][hyh][hxh], f100 = L.sphi[hzh][hyl][hxl], f101 = L.sphi[hzh][hyl][hxh],
                    f110 = L.sphi[hzh][hyh][hxl], f111 = L.sphi[hzh][hyh][hxh];
            const T sx = T(1) - bx.t, sy = T(1) - by.t, sz = T(1) - bz.t;
            const T phi_p = sz * (sy * (sx * f000 + bx.t * f001) + by.t * (sx * f010 + bx.t * f011)) +
                            bz.t * (sy * (sx * f100 + bx.t * f101) + by.t * (sx * f110 + bx.t * f111));
            if (std::is_same<T, float>::value && phi_p > (T)a.phi_fp64) {
                // FP64 weights from the same positions; the cancellation in 1 - phi is exact
                const double gx = (double)q.x * (double)g.sb[0] - 0.5, gy = (double)q.y * (double)g.sb[1] - 0.5,
                             gz = (double)q.z * (double)g.sb[2] - 0.5;
                const double tx = gx - floor(gx), ty = gy - floor(gy), tz = gz - floor(gz);
                const double ux = 1.0 - tx, uy = 1.0 - ty, uz = 1.0 - tz;
                const double ph =
                    uz * (uy * (ux * (double)f000 + tx * (double)f001) + ty * (ux * (double)f010 + tx * (double)f011)) +
                    tz * (uy * (ux * (double)f100 + tx * (double)f101) + ty * (ux * (double)f110 + tx * (double)f111));
                s.w = (T)(1.0 - ph);
            } else {
                s.w = T(1) - phi_p;
            }
        } else {
            const int ix = cell_axis(q.x, g.sb[0], g.nb[0]), iy = cell_axis(q.y, g.sb[1], g.nb[1]),
                      iz = cell_axis(q.z, g.sb[2], g.nb[2]);
            s.w = T(1) - L.sphi[iz - oz + 1][iy - oy + 1][ix - ox + 1];
        }
        a.uf4[p] = s;
    }
}

// One workgroup per brick, or where there are few bricks of many particles
// (gridDim.y = 1 otherwise) several that fill the same brick and share its
// particles: a batch of 512 is a chain of dependent loads (10,000 particles in 8
// bricks, FP64: 14 us with one workgroup each, 10 with three; 65,000 53 and 13).  They
// share while that gives at most two workgroups per compute unit (400,000 in 32^3 FP64
// cells, 1024 bricks: 28 us; sharing up to eight per unit 38; 200,000 in 24^3, 216
// bricks, where two share one: 20, alone 17).
template <typename T, int R, int SM, int HALVES>
__global__ __launch_bounds__(kBrickThreads<HALVES>, (BrickWaves<T, HALVES>::value)) void k_restrict_brick(
    StepArgs<T> a, BrickGrid<T> bg) {
    static_assert(R <= 4, "one thread per fine child plane");
    static_assert(kBrickRows <= kBrickFill, "one particle row per thread");
    __shared__ BrickLds<T, R> L;
    int ox, oy, oz;
    bg.origin(xcd_tile(blockIdx.x, gridDim.x), ox, oy, oz);
    brick_fill<T, R, SM, HALVES>(a, L, threadIdx.x, ox, oy, oz, blockIdx.y == 0);
    __syncthreads();
    brick_particles<T, R>(a, L, threadIdx.x, kBrickThreads<HALVES>, blockIdx.y, gridDim.y, ox, oy, oz);
}

template <typename T, int R> int64_t brick_blocks(const Geo<T> &g) {
    return (int64_t)((g.nb[0] + kBrickX - 1) / kBrickX) * ((g.nb[1] + kBrickY - 1) / kBrickY) *
           ((g.nb[2] + kBrickZ - 1) / kBrickZ);
}

// Sampling for the bulk-velocity and given-velocity sources (sorted order).
template <typename T>
__global__ __launch_bounds__(kBlock) void k_sample(StepArgs<T> a) {
    const int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (i < a.n) {
        const int64_t idx[1] = {i};
        sample_particles<T, 1>(idx, a);
    }
}

// ---------------------------------------------------------------------------
// Drag and advection, one thread per particle in input order (coalesced).
//   F = beta (u_f - u_p), beta written as
//   1/2 rho_f (pi d^2/4) eps*^(2-chi) (0.63 sqrt|u_r| + 4.8 sqrt(mu_f/(rho_f eps* d)))^2
// which equals 1/2 C_D rho_f A eps*^(2-chi) |u_r| with C_D = (0.63 + 4.8/sqrt(Re))^2,
// Re = rho_f eps* d |u_r| / mu_f, chi = 3.7 - 0.65 exp(-(1.5 - log10 Re)^2 / 2), and
// stays finite as |u_r| -> 0 (where F = 0).
// ---------------------------------------------------------------------------
template <typename T>
__global__ __launch_bounds__(kBlock) void k_drag(StepArgs<T> a) {
    __shared__ double red[kWavesPerBlock];
    const Geo<T> &g = a.g;
    const int64_t p = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    double acc[9] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0};   // sum F (3), clamped, V_p, beta, beta u_p (3)
    if (p < a.n) {
        int o = 0;
        const T xs[3] = {clamp_coord(a.pos[3 * p + 0], g.L[0], o), clamp_coord(a.pos[3 * p + 1], g.L[1], o),
                         clamp_coord(a.pos[3 * p + 2], g.L[2], o)};
        const T us[3] = {a.vel[3 * p + 0], a.vel[3 * p + 1], a.vel[3 * p + 2]};
        const T d = a.diam[p];
        const vec4<T> s = a.uf4[p];
        T uf[3] = {s.x, s.y, s.z};
        if (a.vel_source == 2)
            for (int k = 0; k < 3; ++k) uf[k] = a.uf_given[3 * p + k];
        if (a.uf_out)
            for (int k = 0; k < 3; ++k) a.uf_out[3 * p + k] = uf[k];
        const T ur0 = uf[0] - us[0], ur1 = uf[1] - us[1], ur2 = uf[2] - us[2];
        const T mag = dsqrt(ur0 * ur0 + ur1 * ur1 + ur2 * ur2);
        T e = s.w;
        int clamped = 0;
        if (e < a.eps_min) {
            e = a.eps_min;
            clamped = 1;
        }
        // fluid density and viscosity at the particle: fluid 1's, or with the
        // two-fluid drag the mixture by the liquid fraction interpolated from
        // the restricted alpha
        T rho = a.rho_f, mu = a.mu_f;
        if (a.vof) {
            const Axis<T> bx = cic_axis(xs[0], g.sb[0], g.nb[0]);
            const Axis<T> by = cic_axis(xs[1], g.sb[1], g.nb[1]);
            const Axis<T> bz = cic_axis(xs[2], g.sb[2], g.nb[2]);
            const T al = trilin_alpha8(a.alpha8, bx, by, bz, g.nb);
            rho = a.rho_f * al + a.rho_f2 * (T(1) - al);
            mu = a.mu_f * al + a.mu_f2 * (T(1) - al);
        }
        T chi = T(3.7);
        if (mag > T(0)) {
            const T re = rho * e * d * mag / mu;
            const T l = T(1.5) - dlog10(re);
            chi = T(3.7) - T(0.65) * dexp(-l * l * T(0.5));
        }
        const T vfac = dpow(e, T(2) - chi);
        const T sq = T(0.63) * dsqrt(mag) + T(4.8) * dsqrt(mu / (rho * e * d));
        const T area = T(kPi / 4.0) * d * d;
        const T beta = T(0.5) * rho * area * vfac * (sq * sq);
        const T Fs[3] = {beta * ur0, beta * ur1, beta * ur2};
        for (int k = 0; k < 3; ++k) a.drag[3 * p + k] = Fs[k];
        if (a.beta) a.beta[p] = beta;
        for (int k = 0; k < 3; ++k) acc[k] = (double)Fs[k];
        acc[3] = clamped;
        const double dd = (double)d;
        acc[4] = kPi * dd * dd * dd / 6.0;
        if (a.semi) {
            // (beta, beta u_p) with the velocity the drag used, for the
            // semi-implicit deposition (this thread has read uf4[p] already)
            vec4<T> b;
            b.x = beta;
            b.y = beta * us[0];
            b.z = beta * us[1];
            b.w = beta * us[2];
            a.uf4[p] = b;
            acc[5] = (double)beta;
            acc[6] = (double)b.y;
            acc[7] = (double)b.z;
            acc[8] = (double)b.w;
        }

        if (a.advect) {
            // explicit Euler from the old state, specular reflection at the walls
            const T m = a.rho_p * (T(kPi / 6.0) * d * d * d);
            for (int k = 0; k < 3; ++k) {
                T xn = dfma(a.dt, us[k], xs[k]);
                T un = dfma(a.dt, Fs[k] / m, us[k]);
                const T L = g.L[k];
                if (xn < T(0)) {
                    xn = -xn;
                    un = -un;
                } else if (xn > L) {
                    xn = T(2) * L - xn;
                    un = -un;
                }
                xn = fmin(fmax(xn, T(0)), L);
                a.pos[3 * p + k] = xn;
                a.vel[3 * p + k] = un;
            }
        }
    }
    const int slots[9] = {SL_FP, SL_FP + 1, SL_FP + 2, SL_NCLAMP, SL_VTOT, SL_KP, SL_KUP, SL_KUP + 1, SL_KUP + 2};
    const int nsl = a.semi ? 9 : 5;   // uniform over the launch
    for (int k = 0; k < nsl; ++k) {
        const double t = block_sum(acc[k], red);
        if (threadIdx.x == 0) a.part[slots[k] * a.part_stride + blockIdx.x] = t;
    }
}

// ---------------------------------------------------------------------------
// Prolongation bulk -> fine (conservative trilinear)
// ---------------------------------------------------------------------------
// Child l of a parent cell sits at offset o = (l + 1/2)/R - 1/2 (in bulk cell
// units) from the parent centre; its 1-D trilinear weights on the nodes
// (c-1, c, c+1) are (max(-o,0), 1-|o|, max(o,0)).
template <int R> struct ChildW {
    static constexpr double off(int l) { return (l + 0.5) / R - 0.5; }
    static constexpr double w(int l, int k) {  // k = 0,1,2 for c-1, c, c+1
        return k == 0 ? (off(l) < 0 ? -off(l) : 0.0)
                      : (k == 1 ? 1.0 - (off(l) < 0 ? -off(l) : off(l)) : (off(l) > 0 ? off(l) : 0.0));
    }
    static constexpr double mean(int k) {       // (1/R) sum_l w(l, k)
        double s = 0.0;
        for (int l = 0; l < R; ++l) s += w(l, k);
        return s / R;
    }
};

template <typename T, int R>
__device__ __forceinline__ T wsum3(int l, T a0, T a1, T a2) {
    // sum_k w(l,k) a_k, skipping structurally zero weights
    T s = T(ChildW<R>::w(l, 1)) * a1;
    if (ChildW<R>::w(l, 0) != 0.0) s = dfma(T(ChildW<R>::w(l, 0)), a0, s);
    if (ChildW<R>::w(l, 2) != 0.0) s = dfma(T(ChildW<R>::w(l, 2)), a2, s);
    return s;
}

// The bulk fields a prolongation launch transfers (blockIdx.y), their fine
// outputs and the diagnostic slots of their fine sums; field 0 is the solid
// fraction, prolonged as the porosity 1 - phi.
constexpr int kMaxProlong = 8;
template <typename T> struct ProlongSet {
    const T *B[kMaxProlong];
    T *out[kMaxProlong];
    int slot[kMaxProlong];
};

// The fine-grid writes bound this kernel, and the rate of writing depends on
// which addresses are written together: bare 16-byte stores over 512 x 512 x
// 1024 fine cells run at 6.7 TB/s in address order; a workgroup that writes the
// r planes of a tile of 64 x 4 bulk cells, sixteen tiles to an XCD at a time,
// reaches 5.5 TB/s, with the planes one after the other, tiles of 128 x 2 and
// whole layers to an XCD 6.1 TB/s.  (One plane per workgroup reaches 6.5 TB/s
// but interpolates along x and y once per plane: its arithmetic then bounds it.)
//
// A work item is a tile of 256 bulk cells of one layer, 2^xs wide, or where
// that leaves few workgroups one fine plane of such a tile; one launch takes
// every field (blockIdx.y).  The tile's 3 x 3 x 3 neighbourhoods (the tile with a
// one-cell halo, indices clamped at the walls) are staged in LDS in one memory
// round trip, and each thread writes its cell's children plane by plane (ratio 1, a
// copy, stages nothing: eight fields of 4.2 million cells 180 -> 136 us).
// Workgroups loop over the items (prolong_blocks).
constexpr int kPMaxX = 7, kPMinX = 4;   // tiles of 128 x 2 ... 16 x 16 cells
constexpr int kPStage = ((1 << kPMaxX) + 2) * ((kBlock >> kPMaxX) + 2);   // staged values of the widest tile
static_assert(((1 << kPMinX) + 2) * ((kBlock >> kPMinX) + 2) <= kPStage, "the widest tile has the most halo");

// Tile width.  In general the widest that pads x by at most a quarter, else the
// widest of those that pad it least: padding costs idle lanes (3 x 300 x 300 cells of
// ratio 2 take 36 us in tiles of 16 x 16, 163 in 64 x 4), narrow tiles short rows
// (100^3 cells of ratio 2 take 45 us in 16 x 16, where a quarter draws the line, and 36
// in 64 x 4; 72^3 17.6 and 21.2).
//   The writes of ratio 4 bound it whatever is padded, if there are enough tiles, and
// are fastest from rows of 64 cells or 128: FP32 150 x 90 x 50 cells take 202 us in 32
// x 8, 178 in 64 x 4; FP64 72^3 290 in 16 x 16, 208 in 64 x 4, 16 x 64 x 64 62 and 32
// (128 x 2 where x is not a multiple of it: 72^3 294; where it is, 128 x 64 x 64 456, in
// 64 x 4 472).  Up to sixteen cells in FP32, eight in FP64, are the faster in 16 x 16 (16
// x 64 x 64, 17 and 20; 8 x 64 x 64, 28 and 32), and so are few tiles (FP64 32^3: 24 in
// 32 x 8, 29).
static int prolong_shift(const int nb[3], int ratio, bool fp64) {
    const int nx = nb[0];
    auto padded = [&](int xs) { return (((int64_t)nx + (1 << xs) - 1) >> xs) << xs; };
    if (ratio == 4 && nx > (fp64 ? 8 : 16) && (padded(6) >> 6) * (((int64_t)nb[1] + 3) / 4) * nb[2] >= 512)
        return (fp64 ? nx % 128 == 0 : 4 * padded(7) <= 5 * (int64_t)nx) ? 7 : 6;
    for (int xs = kPMaxX; xs >= kPMinX; --xs)
        if (4 * padded(xs) <= 5 * (int64_t)nx) return xs;
    for (int xs = kPMaxX; xs > kPMinX; --xs)
        if (padded(xs) == padded(kPMinX)) return xs;
    return kPMinX;
}
// How a prolongation is split: tile width 2^xs, fine planes per item (all r of them,
// x and y interpolated once, or one where whole tiles would leave the four or more
// fields fewer than 1024 workgroups: FP64 8^3 cells of ratio 4 take 6.9 us a plane at a
// time, 7.4 otherwise, 16^3 8.3 and 9.0; FP32 differs by less, 24^3 10.0 and 8.8),
// items.
struct ProlongSplit {
    int xs, planes;
    int64_t items;
};
static ProlongSplit prolong_split(const int nb[3], int ratio, bool fp64) {
    ProlongSplit p;
    p.xs = prolong_shift(nb, ratio, fp64);
    const int ys = 8 - p.xs;
    const int64_t tiles = (((int64_t)nb[0] + (1 << p.xs) - 1) >> p.xs) * (((int64_t)nb[1] + (1 << ys) - 1) >> ys) * nb[2];
    p.planes = tiles * 4 < 1024 ? 1 : ratio;
    p.items = tiles * (ratio / p.planes);
    return p;
}
static_assert(kBlock == 256, "a tile has 2^8 cells");

// Workgroups per field, one FP64 partial each: one per item, or the most there may be
// (a multiple of the XCDs, so that each keeps its share of the items).
static int64_t prolong_blocks(int64_t n, int64_t ncell, int64_t items) {
    const int64_t most = most_partials(n, ncell);
    return items <= most ? items : most / 8 * 8;
}

template <typename T, int R>
__global__ __launch_bounds__(kBlock) void k_prolong(StepArgs<T> a, ProlongSet<T> fs, int xs, int planes, int64_t items) {
    __shared__ T sb[3][kPStage];
    __shared__ double red[kWavesPerBlock];
    const Geo<T> &g = a.g;
    const int f = blockIdx.y, ys = 8 - xs;
    const int W = 1 << xs, H = 1 << ys, pitch = W + 2;
    const T *__restrict__ B = fs.B[f];
    T *__restrict__ out = fs.out[f];
    const int tnx = (g.nb[0] + W - 1) >> xs, tny = (g.nb[1] + H - 1) >> ys;
    const int64_t layer = (int64_t)tnx * tny;
    const int64_t nx = g.nb[0], nxy = (int64_t)g.nb[0] * g.nb[1];
    const int64_t nfx = g.nf[0], nfxy = (int64_t)g.nf[0] * g.nf[1];
    const int i = (int)threadIdx.x & (W - 1), j = (int)threadIdx.x >> xs;
    double sum = 0.0;
    for (int64_t it = blockIdx.x; it < items; it += gridDim.x) {
        const int64_t item = xcd_tile(it, items, layer < kXcdChunk ? kXcdChunk : layer);
        const uint32_t trow = (uint32_t)item / (uint32_t)tnx, tlay = trow / (uint32_t)tny;   // fewer than 2^31 items
        const int cx0 = (int)((uint32_t)item - trow * (uint32_t)tnx) << xs, cy0 = (int)(trow - tlay * (uint32_t)tny) << ys;
        const int pz = (int)tlay * planes, cz = pz / R, lz0 = pz % R;   // first fine plane
        if constexpr (R == 1) {   // the child is the cell (a sum with the defect 0)
            const int cx = cx0 + i, cy = cy0 + j;
            if (cx < g.nb[0] && cy < g.nb[1]) {
                const int64_t c = cz * nxy + cy * nx + cx;
                const T q = (f == 0 ? T(1) - B[c] : B[c]) + T(0);
                store_row<T, 1>(out + c, &q);
                if (c >= a.own_c0 && c < a.own_c1) sum += (double)q;
            }
            continue;
        }
        // staging: the H + 2 rows of the tile in two rounds of H, and the two
        // halo columns, every load issued before the first LDS write
        const int64_t zo[3] = {(cz > 0 ? cz - 1 : 0) * nxy, cz * nxy, (cz + 1 < g.nb[2] ? cz + 1 : cz) * nxy};
        const int si[3] = {i + 1, i + 1, (threadIdx.x & 1) ? W + 1 : 0};
        const int sj[3] = {j, j + H, (int)threadIdx.x >> 1};
        const bool on[3] = {true, j < 2, (int)threadIdx.x < 2 * (H + 2)};
        T v[3][3];
#pragma unroll
        for (int u = 0; u < 3; ++u) {
            const int64_t o = clampi(cy0 - 1 + sj[u], g.nb[1]) * nx + clampi(cx0 - 1 + si[u], g.nb[0]);
            if (on[u])
#pragma unroll
                for (int k = 0; k < 3; ++k) v[u][k] = B[zo[k] + o];
        }
#pragma unroll
        for (int u = 0; u < 3; ++u)
            if (on[u])
#pragma unroll
                for (int k = 0; k < 3; ++k) sb[k][sj[u] * pitch + si[u]] = f == 0 ? T(1) - v[u][k] : v[u][k];
        __syncthreads();
        const int cx = cx0 + i, cy = cy0 + j;
        if (cx < g.nb[0] && cy < g.nb[1]) {
            T b[3][3][3];
#pragma unroll
            for (int k = 0; k < 3; ++k)
#pragma unroll
                for (int r = 0; r < 3; ++r)
#pragma unroll
                    for (int c = 0; c < 3; ++c) b[k][r][c] = sb[k][(j + r) * pitch + i + c];
            // defect of the parent: B_c - (1/R^3) sum of the trilinear children
            T D = T(0);
            if constexpr (R > 1) {
                T mz[3];
#pragma unroll
                for (int k = 0; k < 3; ++k) {
                    T my[3];
#pragma unroll
                    for (int r = 0; r < 3; ++r)
                        my[r] = T(ChildW<R>::mean(0)) * b[k][r][0] + T(ChildW<R>::mean(1)) * b[k][r][1] +
                                T(ChildW<R>::mean(2)) * b[k][r][2];
                    mz[k] = T(ChildW<R>::mean(0)) * my[0] + T(ChildW<R>::mean(1)) * my[1] +
                            T(ChildW<R>::mean(2)) * my[2];
                }
                T mean = T(ChildW<R>::mean(0)) * mz[0] + T(ChildW<R>::mean(1)) * mz[1] +
                         T(ChildW<R>::mean(2)) * mz[2];
                D = b[1][1][1] - mean;
            }
            // separable trilinear: x, then y (every child row), then z plane by
            // plane, each plane's rows stored together
            T Y[R][3][R];
#pragma unroll
            for (int k = 0; k < 3; ++k) {
                T X[3][R];
#pragma unroll
                for (int r = 0; r < 3; ++r)
#pragma unroll
                    for (int lx = 0; lx < R; ++lx) X[r][lx] = wsum3<T, R>(lx, b[k][r][0], b[k][r][1], b[k][r][2]);
#pragma unroll
                for (int ly = 0; ly < R; ++ly)
#pragma unroll
                    for (int lx = 0; lx < R; ++lx) Y[ly][k][lx] = wsum3<T, R>(ly, X[0][lx], X[1][lx], X[2][lx]);
            }
            T *__restrict__ o = out + (int64_t)R * cz * nfxy + (int64_t)R * cy * nfx + (int64_t)R * cx;
            double s = 0.0;
#pragma unroll
            for (int lz = 0; lz < R; ++lz) {
                if (lz < lz0 || lz >= lz0 + planes) continue;   // uniform over the workgroup
#pragma unroll
                for (int ly = 0; ly < R; ++ly) {
                    T q[R];
#pragma unroll
                    for (int lx = 0; lx < R; ++lx) {
                        q[lx] = wsum3<T, R>(lz, Y[ly][0][lx], Y[ly][1][lx], Y[ly][2][lx]) + D;
                        s += (double)q[lx];
                    }
                    store_row<T, R>(o + lz * nfxy + ly * nfx, q);
                    // keeps the scheduler from computing every row before the
                    // first store (all r^3 values live at once)
                    __builtin_amdgcn_sched_barrier(0);
                }
            }
            const int64_t c = cz * nxy + cy * nx + cx;   // owned cells enter the fine-grid sums
            if (c >= a.own_c0 && c < a.own_c1) sum += s;
        }
        if (it + gridDim.x < items) __syncthreads();   // the stage is used again (uniform over the workgroup)
    }
    const double t = block_sum(sum, red);
    if (threadIdx.x == 0) a.part[fs.slot[f] * a.part_stride + blockIdx.x] = t;
}

// ---------------------------------------------------------------------------
// Final fixed-order reduction of the per-workgroup partials
// ---------------------------------------------------------------------------
struct DiagSpec {
    int nblk[SL_COUNT];
    double scale[SL_COUNT];
};

// One workgroup per slot: thread t takes the partials t, t + kDiagThreads, ... in
// order, kDiagBatch loads in flight, then a fixed tree.  Deterministic.  Bound by
// the launch and by one or (39,000 partials of 10 million particles) five memory
// round trips; a stage of many chunks and one that combines them were two
// launches (2.8 + 2.5 us of a small step, 4.9 + 4.7 of one of 2 million particles;
// in one 2.9 and 4.7, and 10.7 for 10 million instead of 9.7 and the gap).
constexpr int kDiagThreads = 1024, kDiagBatch = 8;

__global__ __launch_bounds__(kDiagThreads) void k_diag(const double *__restrict__ part, int64_t ps, DiagSpec spec,
                                                       double *__restrict__ diag) {
    __shared__ double red[kDiagThreads / kWave];
    const int s = blockIdx.x;
    const bool is_max = (s == SL_MAXPHI);
    const int nb = spec.nblk[s];
    const double *src = part + s * ps;
    double v = 0.0;
    for (int j0 = threadIdx.x; j0 < nb; j0 += kDiagBatch * kDiagThreads) {
        double x[kDiagBatch];
#pragma unroll
        for (int u = 0; u < kDiagBatch; ++u) {
            const int j = j0 + u * kDiagThreads;
            x[u] = src[j < nb ? j : nb - 1];
        }
#pragma unroll
        for (int u = 0; u < kDiagBatch; ++u) {
            const double y = j0 + u * kDiagThreads < nb ? x[u] : 0.0;
            v = is_max ? fmax(v, y) : v + y;
        }
    }
    v = is_max ? wave_max(v) : wave_sum(v);
    if (threadIdx.x % kWave == 0) red[threadIdx.x / kWave] = v;
    __syncthreads();
    if (threadIdx.x == 0) {
        double t = 0.0;
        for (int w = 0; w < kDiagThreads / kWave; ++w) t = is_max ? fmax(t, red[w]) : t + red[w];
        diag[s] = t * spec.scale[s];
    }
}

// ---------------------------------------------------------------------------
// Host dispatch
// ---------------------------------------------------------------------------
// Restriction of fields F0 .. F1 - 1: four threads per cell for r = 4, one
// otherwise.
template <typename T, int R, int SM, int F0, int F1> static void restrict_fields(const StepArgs<T> &a, hipStream_t st) {
    if constexpr (R == 4)
        hipLaunchKernelGGL((k_restrict_planes<T, SM, F0, F1, false>),
                           dim3((unsigned)((a.g.ncell + kPlaneCells - 1) / kPlaneCells)), dim3(kBlock), 0, st, a);
    else
        hipLaunchKernelGGL((k_restrict<T, R, SM, F0, F1>), dim3((unsigned)((a.g.ncell + kBlock - 1) / kBlock)),
                           dim3(kBlock), 0, st, a);
}

template <typename T, int R, int SM>
static void launch_grid_stages(const StepArgs<T> &a, hipStream_t st, int phases) {
    const int64_t cb = (a.g.ncell + kBlock - 1) / kBlock;
    const int64_t pb = (a.n + kBlock - 1) / kBlock;
    const int64_t nc = a.g.ncell, nf = a.g.nfine;
    if (phases & kPhaseVelocity) {
    if (a.vel_source == 0) {
        // the pressure (for the gradient only), then u, v, w with the lookup
        a.mk->mark("restrict_p", st);
        restrict_fields<T, R, SM, 3, 4>(a, st);
        a.mk->mark("restrict_lookup", st);
        const int64_t nbk = brick_blocks<T, R>(a.g);
        const BrickGrid<T> bg{(a.g.nb[0] + kBrickX - 1) / kBrickX, (a.g.nb[1] + kBrickY - 1) / kBrickY};
        auto bricks = [&](auto hc) {
            constexpr int H = decltype(hc)::value;
            // bricks alone that fill the chip take one workgroup each; fewer share the
            // mean number of particles in batches
            const int64_t batch = nbk * kBrickThreads<H>;
            const int64_t parts = std::max<int64_t>(1, std::min<int64_t>(kBrickFew / nbk, (a.n + batch - 1) / batch));
            hipLaunchKernelGGL((k_restrict_brick<T, R, SM, H>), dim3((unsigned)nbk, (unsigned)parts),
                               dim3(kBrickThreads<H>), 0, st, a, bg);
        };
        if (R == 4 || nbk <= kBrickFew) bricks(std::integral_constant<int, 2>{});
        else bricks(std::integral_constant<int, R == 4 ? 2 : 1>{});
    } else if (a.vel_source == 3) {
        if constexpr (std::is_same<T, float>::value) {
            a.mk->mark("restrict", st);
            restrict_fields<T, R, SM, 0, 4>(a, st);
            a.mk->mark("mlp_pack", st);
            launch_mlp_pack(a, st);
            if (a.n > 0) {
                a.mk->mark("mlp_infer", st);
                launch_mlp_infer(a, st);
                a.mk->mark("mlp_check", st);
                launch_mlp_check(a, st);
            }
        }
    } else {
        a.mk->mark("restrict", st);
        restrict_fields<T, R, SM, 0, 4>(a, st);
        if (a.n > 0) a.mk->mark("sample", st);
        if (a.n > 0) hipLaunchKernelGGL(k_sample<T>, dim3(pb), dim3(kBlock), 0, st, a);
    }
    if (a.vof) {
        a.mk->mark("restrict_alpha", st);
        if constexpr (R == 4)
            hipLaunchKernelGGL((k_restrict_planes<T, SM, 0, 1, true>), dim3((unsigned)((nc + kPlaneCells - 1) / kPlaneCells)),
                               dim3(kBlock), 0, st, a);
        else
            hipLaunchKernelGGL((k_restrict_alpha<T, R, SM>), dim3(cb), dim3(kBlock), 0, st, a);
        if (a.n > 0) a.mk->mark("pack_alpha", st);
        if (a.n > 0) hipLaunchKernelGGL(k_pack_alpha8<T>, dim3(cb), dim3(kBlock), 0, st, a);
    }
    if (a.n > 0) a.mk->mark("drag", st);
    if (a.n > 0) hipLaunchKernelGGL(k_drag<T>, dim3(pb), dim3(kBlock), 0, st, a);
    }
    if (phases & kPhaseSource) {
    a.mk->mark("deposit_force", st);
    launch_deposit_force<T, SM>(a, st);
    if (a.semi) {
        a.mk->mark("deposit_semi", st);
        launch_deposit_semi<T, SM>(a, st);
    }
    }
    if (phases & kPhaseProlong) {
    ProlongSet<T> fs;
    int m = 0;
    auto add = [&](const T *B, T *out, int slot) {
        fs.B[m] = B;
        fs.out[m] = out;
        fs.slot[m++] = slot;
    };
    add(a.phi, a.fine_eps, SL_EPSF);
    for (int k = 0; k < 3; ++k) add(a.F + k * nc, a.fine_F + k * nf, SL_FF + k);
    if (a.semi) {
        add(a.K, a.fine_K, SL_KF);
        for (int k = 0; k < 3; ++k) add(a.KU + k * nc, a.fine_KU + k * nf, SL_KUF + k);
    }
    a.mk->mark("prolong", st);
    const ProlongSplit ps = prolong_split(a.g.nb, R, sizeof(T) == 8);
    hipLaunchKernelGGL((k_prolong<T, R>), dim3((unsigned)prolong_blocks(a.n, nc, ps.items), (unsigned)m), dim3(kBlock), 0,
                       st, a, fs, ps.xs, ps.planes, ps.items);
    }
}

template <typename T, int SM> static void launch_by_ratio(const StepArgs<T> &a, hipStream_t st, int phases) {
    switch (a.ratio) {
    case 1: launch_grid_stages<T, 1, SM>(a, st, phases); break;
    case 2: launch_grid_stages<T, 2, SM>(a, st, phases); break;
    default: launch_grid_stages<T, 4, SM>(a, st, phases); break;
    }
}

template <typename T> hipError_t launch_stages(const StepArgs<T> &a, hipStream_t st, int phases) {
    const int64_t cb = (a.g.ncell + kBlock - 1) / kBlock;
    const int64_t pb = (a.n + kBlock - 1) / kBlock;
    const int sm = a.sum_mode;   // FP32 modes; the FP64 mode sums plainly

    // workgroups per diagnostic slot (each writes one partial per slot), checked
    // against the partials' stride before anything is launched
    DiagSpec spec;
    for (int s = 0; s < SL_COUNT; ++s) {
        spec.nblk[s] = (int)cb;
        spec.scale[s] = 1.0;
    }
    const int db = deposit_blocks(a.n, a.g.ncell, a.cic);
    spec.nblk[SL_PHISUM] = db;
    spec.nblk[SL_MAXPHI] = db;
    for (int k = 0; k < 3; ++k) spec.nblk[SL_FB + k] = db;
    spec.nblk[SL_VTOT] = a.n > 0 ? (int)pb : 0;
    spec.nblk[SL_NOUT] = a.n > 0 ? a.bin_tiles : 0;
    const int npart = a.n > 0 ? (int)pb : 0;   // k_drag
    for (int k = 0; k < 3; ++k) spec.nblk[SL_FP + k] = npart;
    spec.nblk[SL_NCLAMP] = npart;
    const int nmlp = (a.vel_source == 3 && a.n > 0) ? (int)mlp_check_blocks(a.n_bricks) : 0;
    spec.nblk[SL_NFALL] = nmlp;
    spec.nblk[SL_MLPERR] = nmlp;
    spec.nblk[SL_MLPREF] = nmlp;
    spec.nblk[SL_MLPSAMP] = nmlp;
    const int ptiles =   // k_prolong
        (int)prolong_blocks(a.n, a.g.ncell, prolong_split(a.g.nb, a.ratio, sizeof(T) == 8).items);
    spec.nblk[SL_EPSF] = ptiles;
    for (int k = 0; k < 3; ++k) spec.nblk[SL_FF + k] = ptiles;
    for (int k = 0; k < 4; ++k) {
        spec.nblk[SL_KP + k] = a.semi ? npart : 0;   // k_drag
        spec.nblk[SL_KB + k] = a.semi ? db : 0;      // deposition
        spec.nblk[SL_KF + k] = a.semi ? ptiles : 0;  // prolongation
        spec.scale[SL_KB + k] = a.g.vb;
        spec.scale[SL_KF + k] = a.g.vf;
    }
    spec.scale[SL_PHISUM] = a.g.vb;
    for (int k = 0; k < 3; ++k) {
        spec.scale[SL_FB + k] = a.g.vb;
        spec.scale[SL_FF + k] = a.g.vf;
    }
    spec.scale[SL_EPSF] = a.g.vf;
    for (int s = 0; s < SL_COUNT; ++s)
        if (spec.nblk[s] > a.part_stride) return hipErrorInvalidValue;   // partials would not fit

    if (phases & kPhaseDeposit) {
        a.mk->mark("deposit_phi", st);
        if constexpr (std::is_same<T, float>::value) {
            if (sm == kSumKahan) launch_deposit_phi<T, kSumKahan>(a, st);
            else if (sm == kSumWide) launch_deposit_phi<T, kSumWide>(a, st);
            else launch_deposit_phi<T, kSumPlain>(a, st);
        } else {
            launch_deposit_phi<T, kSumPlain>(a, st);
        }
    }
    if (phases & (kPhaseVelocity | kPhaseSource | kPhaseProlong)) {
        if constexpr (std::is_same<T, float>::value) {
            if (sm == kSumKahan) launch_by_ratio<T, kSumKahan>(a, st, phases);
            else if (sm == kSumWide) launch_by_ratio<T, kSumWide>(a, st, phases);
            else launch_by_ratio<T, kSumPlain>(a, st, phases);
        } else {
            launch_by_ratio<T, kSumPlain>(a, st, phases);
        }
    }
    if (phases & kPhaseDiag) {
        a.mk->mark("diag", st);
        hipLaunchKernelGGL(k_diag, dim3(SL_COUNT), dim3(kDiagThreads), 0, st, a.part, a.part_stride, spec, a.diag);
        a.mk->mark(nullptr, st);
    }
    return hipGetLastError();
}

template hipError_t launch_stages<float>(const StepArgs<float> &, hipStream_t, int);
template hipError_t launch_stages<double>(const StepArgs<double> &, hipStream_t, int);

}  // namespace cpl
