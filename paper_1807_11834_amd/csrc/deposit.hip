// deposit.hip -- particle -> bulk-cell deposition of the solid volume fraction
// and of the momentum source, deterministic and without atomics.
//
//   phi_c   = sum_p w_pc V_p / V_b                 (porosity eps = 1 - phi)
//   F_fpi,c = -(1/V_b) sum_p w_pc F_p              (counterpart of the drag)
//   K_c     = (1/V_b) sum_p w_pc beta_p            (semi-implicit split of F_fpi:
//   KU_c    = (1/V_b) sum_p w_pc beta_p u_p         F_fpi = -K u_f + KU in uniform flow)
//
// The particles are in the canonical (cell, id) order with CSR offsets `start`.
// CIC: two passes through partial sums per group of source rows (see below);
// every particle is staged once per pass.  NGP: a workgroup sums the segments of a
// group of cells, staged together.
#include <algorithm>
#include <type_traits>

#include "common.hpp"
#include "launch.hpp"

namespace cpl {

constexpr int kChunk = 256;   // particles staged per wave and chunk
static_assert(kChunk % kWave == 0, "a chunk is staged in whole waves");

// What a deposition pass sums: V_p / V_b (phi), the drag F_p (source) or
// (beta_p, beta_p u_p) (semi-implicit split).
enum DepMode { kPhi = 0, kForce = 1, kSemi = 2 };
template <int MODE> struct DepNc { static constexpr int value = MODE == kPhi ? 1 : (MODE == kForce ? 3 : 4); };

template <typename T> __device__ __forceinline__ T sphere_volume(T d) { return T(kPi / 6.0) * d * d * d; }
template <typename T> __device__ __forceinline__ T vol_over_vb(T d, T inv_vb) { return sphere_volume(d) * inv_vb; }

// Bulk pressure gradient of cell c written to G ([3][ncell]), in the arithmetic
// of gradient_at(): the cell's and its six neighbours' (hi, lo) pressure are
// loaded first, unconditionally (a neighbour beyond a wall is the cell itself),
// so that a kernel can issue these loads with its others and wait once.
template <typename T> struct GradLoads {
    T hi[7], lo[7];   // centre, then (low, high) neighbour per axis
};

template <typename T>
__device__ __forceinline__ GradLoads<T> load_gradient(int64_t c, int cx, int cy, int cz, const Geo<T> &g,
                                                      const T *__restrict__ P, const T *__restrict__ Plo) {
    const int idx[3] = {cx, cy, cz};
    const int64_t stride[3] = {1, g.nb[0], (int64_t)g.nb[0] * g.nb[1]};
    GradLoads<T> r;
    r.hi[0] = P[c];
    r.lo[0] = Plo[c];
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        const int64_t kl = idx[a] > 0 ? c - stride[a] : c, kh = idx[a] < g.nb[a] - 1 ? c + stride[a] : c;
        r.hi[1 + 2 * a] = P[kl];
        r.lo[1 + 2 * a] = Plo[kl];
        r.hi[2 + 2 * a] = P[kh];
        r.lo[2 + 2 * a] = Plo[kh];
    }
    return r;
}

template <typename T>
__device__ __forceinline__ void write_gradient(const GradLoads<T> &v, int64_t c, int cx, int cy, int cz,
                                               const Geo<T> &g, T *__restrict__ G) {
    const int idx[3] = {cx, cy, cz};
    const double p0 = (double)v.hi[0] + (double)v.lo[0];
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        const double pl = (double)v.hi[1 + 2 * a] + (double)v.lo[1 + 2 * a];
        const double ph = (double)v.hi[2 + 2 * a] + (double)v.lo[2 + 2 * a];
        const int nax = g.nb[a];
        const double h = (double)g.hb[a];
        double gr;
        if (nax == 1) gr = 0.0;
        else if (idx[a] == 0) gr = (ph - p0) / h;
        else if (idx[a] == nax - 1) gr = (p0 - pl) / h;
        else gr = (ph - pl) / (2.0 * h);
        G[a * g.ncell + c] = (T)gr;
    }
}

// The values one particle deposits: V_p / V_b from its record (kPhi), its drag
// (kForce) or (beta_p, beta_p u_p) (kSemi).  The solid fraction comes first in a
// step, so its pass also makes the sorted copy of the particles that the later
// stages read: it takes the record from the input-order copy pk through the
// permutation (a random read that its arithmetic hides) and stores it at the
// sorted position.
template <typename T, int MODE>
__device__ __forceinline__ void load_values(int64_t id, const vec4<T> &q, const T *__restrict__ drag,
                                            const vec4<T> *__restrict__ src4, T inv_vb, T (&val)[DepNc<MODE>::value]) {
    if constexpr (MODE == kForce) {
        for (int c = 0; c < 3; ++c) val[c] = drag[3 * id + c];
    } else if constexpr (MODE == kSemi) {
        const vec4<T> b = src4[id];
        val[0] = b.x;
        val[1] = b.y;
        val[2] = b.z;
        val[3] = b.w;
    } else {
        val[0] = vol_over_vb(q.w, inv_vb);
    }
}

// ---------------------------------------------------------------------------
// NGP (containing cell)
// ---------------------------------------------------------------------------
// A workgroup takes a group of consecutive cells at a time, whose particles are one
// run of the sorted order.  The run passes through LDS in chunks, every load of a
// chunk in flight together; a cell's part of the chunk is then summed in canonical
// order, by lane (cell) of wave (component) or, in a WIDE group of 256 cells, by
// thread (cell) for all components.  One thread per cell that loads and adds
// particle by particle waits for two dependent loads per particle: 512 cells of 20
// particles in FP64 took 3 + 12 us (sorted copy, solid fraction) and 19 us (source),
// on two compute units.  In groups of 64 cells they were two chunks of 8 workgroups
// (10.4 and 10.2 us); in groups of 16, with four of a cell's values read from LDS at
// a time, 6.6 and 6.1.
// A cell's sum of v, or for the solid fraction of v / V_b: the product rounded
// before it is widened, otherwise one FMA with the running sum.
template <typename T, int SM, int MODE> struct NgpSum {
    static constexpr bool kFma = MODE == kPhi && SM != kSumWide;
    typename std::conditional<kFma, FmaSum<T, SM>, CellSum<T, SM>>::type acc;
    __device__ __forceinline__ void add(T v, T inv_vb) {
        if constexpr (kFma) acc.add(v, inv_vb);
        else acc.add(MODE == kPhi ? v * inv_vb : v);
    }
    __device__ __forceinline__ T value() const { return acc.value(); }
};
constexpr int kNgpItems = 4, kNgpChunk = kBlock * kNgpItems, kNgpRead = 4;
// Cells of a group.  With few particles per cell a wide group: three quarters of the
// threads of a group of 64 have no cell to sum, and the groups' barriers are most of
// the time.  Solid fraction and source of 128 x 128 x 256 cells with 0.24 particles
// each take 37 + 67 us so, 78 + 108 in groups of 64; with 1.2, 119 + 126 and 121 + 139;
// with 2.4, 330 + 225 and 227 + 228.  Where a wide group has a particle for every
// second cell or fewer each thread loads its own (20,000 particles in all: 26 + 50
// us; through LDS 29 + 55).
//   Otherwise a cell per lane, or sixteen in up to 8192 cells, where that leaves most
// compute units without a workgroup (4096 cells of 10 particles: 7.5 + 7.4 us, in
// groups of 64 8.1 + 8.0; 13,824 of 11: 11.0 + 10.7 and 9.2 + 9.5), but no more than
// have a chunk of particles: a group's chunks are summed one after the other (64 cells
// of 3125 particles: 123 + 190 us; in groups of sixteen 1572 + 2346, with a thread per
// cell 1027 + 1771).
constexpr int kNgpSparse = 2;     // particles per cell of the widest groups, at most
constexpr int kNgpDirect = 128;   // particles of a wide group that are not staged
static int ngp_cells(int64_t n, int64_t ncell) {
    if (n <= kNgpSparse * ncell) return kBlock;
    int cells = ncell <= 8192 ? 16 : kWave;
    while (cells > 1 && cells * n > kNgpChunk * ncell) cells /= 2;
    return cells;
}

template <typename T, int SM, int MODE, bool WIDE>
__global__ __launch_bounds__(kBlock) void k_deposit_ngp(const int32_t *__restrict__ start,
                                                        const vec4<T> *__restrict__ pk, vec4<T> *__restrict__ sp,
                                                        const int32_t *__restrict__ perm,
                                                        const T *__restrict__ drag, int64_t n, Geo<T> g,
                                                        const T *__restrict__ P, const T *__restrict__ Plo,
                                                        T *__restrict__ out, T *__restrict__ out2, T *__restrict__ G,
                                                        double *__restrict__ part, int64_t ps, int cells) {
    constexpr int NC = DepNc<MODE>::value;
    static_assert(NC <= kWavesPerBlock, "a wave per component");
    constexpr int NA = WIDE ? NC : 1;   // components a thread sums
    __shared__ T val[NC][kNgpChunk];
    __shared__ double red[kWavesPerBlock];
    const int lane = threadIdx.x % kWave, comp = WIDE ? 0 : threadIdx.x / kWave;
    double vsum[NA] = {}, vmax = 0.0;
    for (int64_t c0 = (int64_t)blockIdx.x * cells; c0 < g.ncell; c0 += (int64_t)gridDim.x * cells) {
        const int64_t c = c0 + (WIDE ? (int)threadIdx.x : lane);
        const int64_t c1 = c0 + cells < g.ncell ? c0 + cells : g.ncell;
        const bool mine = c < c1 && comp < NC;
        const int32_t rs = seg_clamp(start[c0], n), re = seg_clamp(start[c1], n);
        int32_t s = 0, e = 0;
        if (mine) {
            s = seg_clamp(start[c], n);
            e = seg_clamp(start[c + 1], n);
        }
        // the gradient, by the wave with no component or in a wide group by every thread
        GradLoads<T> gl;
        int cx = 0, cy = 0, cz = 0;
        const bool grad = MODE == kForce && (WIDE || comp == kWavesPerBlock - 1) && c < c1;
        if (grad) {
            decode_cell(c, g.nb, cx, cy, cz);
            gl = load_gradient(c, cx, cy, cz, g, P, Plo);
        }
        NgpSum<T, SM, MODE> acc[NA];
        // few particles in a wide group: each thread loads its own
        const bool direct = WIDE && re - rs <= kNgpDirect;   // uniform over the workgroup
        if constexpr (WIDE)
            if (direct && mine)
                for (int32_t p = s; p < e; ++p) {
                    int64_t id = perm[p];
                    if (id < 0 || id >= n) id = 0;
                    vec4<T> q;
                    T v[NC];
                    if constexpr (MODE == kPhi) {
                        q = pk[id];
                        sp[p] = q;
                        v[0] = sphere_volume(q.w);
                    } else {
                        load_values<T, MODE>(id, q, drag, pk, g.inv_vb, v);
                    }
#pragma unroll
                    for (int j = 0; j < NA; ++j) acc[j].add(v[j], g.inv_vb);
                }
        for (int64_t cs = direct ? re : rs; cs < re; cs += kNgpChunk) {   // uniform over the workgroup
            const int m = (int)(re - cs < kNgpChunk ? re - cs : kNgpChunk);
            int64_t id[kNgpItems];
            vec4<T> q[kNgpItems];
            T v[kNgpItems][NC];
#pragma unroll
            for (int u = 0; u < kNgpItems; ++u) {
                const int k = (int)threadIdx.x + u * kBlock;
                const int64_t i = perm[cs + (k < m ? k : 0)];
                id[u] = (i < 0 || i >= n) ? 0 : i;   // perm is a permutation of [0, n)
            }
#pragma unroll
            for (int u = 0; u < kNgpItems; ++u) {
                if constexpr (MODE == kPhi) q[u] = pk[id[u]];
                else load_values<T, MODE>(id[u], q[u], drag, pk, g.inv_vb, v[u]);
            }
#pragma unroll
            for (int u = 0; u < kNgpItems; ++u) {
                const int k = (int)threadIdx.x + u * kBlock;
                if (k >= m) continue;
                if constexpr (MODE == kPhi) {
                    sp[cs + k] = q[u];
                    v[u][0] = sphere_volume(q[u].w);
                }
#pragma unroll
                for (int j = 0; j < NC; ++j) val[j][k] = v[u][j];
            }
            __syncthreads();
            if (mine) {
                const int32_t b0 = (int32_t)((s > cs ? s : cs) - cs), b1 = (int32_t)((e < cs + m ? e : cs + m) - cs);
                for (int32_t k = b0; k < b1; k += kNgpRead) {
                    T x[kNgpRead][NA];
#pragma unroll
                    for (int u = 0; u < kNgpRead; ++u)
#pragma unroll
                        for (int j = 0; j < NA; ++j) x[u][j] = val[comp + j][k + u < b1 ? k + u : k];
#pragma unroll
                    for (int u = 0; u < kNgpRead; ++u)
                        if (k + u < b1)
#pragma unroll
                            for (int j = 0; j < NA; ++j) acc[j].add(x[u][j], g.inv_vb);
                }
            }
            __syncthreads();
        }
        if (mine) {
#pragma unroll
            for (int j = 0; j < NA; ++j) {
                const int k = comp + j;
                const T t = acc[j].value();
                const T f = MODE == kPhi ? t : (MODE == kForce ? -t * g.inv_vb : t * g.inv_vb);
                if (MODE != kSemi || k == 0) out[k * g.ncell + c] = f;
                else out2[(k - 1) * g.ncell + c] = f;
                vsum[j] += (double)f;
                if (MODE == kPhi) vmax = fmax(vmax, (double)f);
            }
        }
        if (grad) write_gradient(gl, c, cx, cy, cz, g, G);
    }
#pragma unroll
    for (int j = 0; j < NA; ++j) {
        const int k = comp + j;
        const double t = WIDE ? block_sum(vsum[j], red) : wave_sum(vsum[j]);
        const int slot = MODE == kPhi ? SL_PHISUM : (MODE == kForce ? SL_FB + k : SL_KB + k);
        if ((WIDE ? (int)threadIdx.x : lane) == 0 && k < NC) part[slot * ps + blockIdx.x] = t;
    }
    if constexpr (MODE == kPhi) {
        const double m = WIDE ? block_max(vmax, red) : wave_max(vmax);
        if (threadIdx.x == 0) part[SL_MAXPHI * ps + blockIdx.x] = m;
    }
}
static_assert(SL_KUB == SL_KB + 1, "the semi-implicit sums are consecutive");

// ---------------------------------------------------------------------------
// CIC (trilinear to the 8 nearest bulk cell centres, folded at the walls)
// ---------------------------------------------------------------------------
// Pass 1, k_deposit_rows: one wave per (GS x GS group of source rows in y and
// z, 64-cell x segment), GS = 2 (or 1 on small grids, see deposit_group()).  For
// each source row of its group the wave stages the particles of the source
// cells x0-1 .. x0+64 once (in chunks), with their x-stencil, their weights on
// the three target y-rows and z-rows around the source row and the deposited
// value(s).  Lane x then accumulates, over the particles of source cells x-1,
// x, x+1 in canonical order, the contributions to target cell x of the
// (GS + 2) x (GS + 2) target rows the group reaches (y-rows GS gy - 1 ..
// GS gy + GS, likewise in z), and writes each to the partial slot of its
// (z-group, y-group) offset from the target.
// Pass 2, k_deposit_sum: per target cell, the <= 4 (GS = 2) or <= 9 (GS = 1)
// partials of the source groups it receives from, in ascending (z-group,
// y-group) order.
// With GS = 2 a target row receives from 2 x 2 groups rather than from 3 x 3
// source rows: the partial sums written and read back are 4/9 of one slot per
// source row; GS = 1 trades that for four times the waves.
//
// The staged values of a particle are read by three lanes (its cell's and the
// two neighbours'), each lane at a place of its own.  They are kept as 16-byte
// records, one read for four values.  The pass is bound by its arithmetic (the
// VALU is busy 60 % of the time; LDS bank conflicts are a few percent) and by the
// loads of the particles' drags, a line each in the order of their ids: 248 us for
// the solid fraction of the bed of 10 million and its sorted copy, 264 for the
// source.  Records of fewer words, other chunks and unconditional loads: no gain.
template <typename T, int MODE> struct RowStage {
    vec4<T> wy[kWavesPerBlock][kChunk];   // weights on target rows y'-1, y', y'+1; weight of the upper x node
    vec4<T> wz[kWavesPerBlock][kChunk];   // weights on target layers z'-1, z', z'+1; x nodes lo | hi << 16 (bits)
    // V_p / V_b, F_p (and a word unused), or (beta_p, beta_p u_p)
    typename std::conditional<MODE == kPhi, T, vec4<T>>::type val[kWavesPerBlock][kChunk];
};

__device__ __forceinline__ float as_value(int32_t b, float) { return __int_as_float(b); }
__device__ __forceinline__ double as_value(int32_t b, double) { return __longlong_as_double((long long)b); }
__device__ __forceinline__ int32_t as_bits(float v) { return __float_as_int(v); }
__device__ __forceinline__ int32_t as_bits(double v) { return (int32_t)__double_as_longlong(v); }

// Row-pass sums s += w v under the step's sum mode: FP32 with Kahan
// compensation (the product w v formed by an FMA against the running
// compensation, so the term is rounded once), FP32 plainly, or widened to FP64
// registers with one FMA per term (both products exact in FP64: every term is
// rounded once at FP64 precision; FP64 FMAs issue at the rate of unpacked FP32
// ones on this chip).  The FP64 mode sums with plain FP64 FMAs (the at most ~100
// terms of a partial sum carry an error below 1e-14 of their magnitudes).
template <typename T, int SM> using RowSum = FmaSum<T, SM>;

template <typename T>
__device__ __forceinline__ void row_weights(const Axis<T> &a, int c, T w[3]) {
    for (int j = 0; j < 3; ++j) {
        const int t = c - 1 + j;
        T v = T(0);
        if (a.lo == t) v += T(1) - a.t;
        if (a.hi == t) v += a.t;
        w[j] = v;
    }
}

// Lowest source group (of G rows) that reaches target row t: floor((t - 1) / G)
// (-1 for t = 0).
template <int G> __device__ __forceinline__ int group_lo(int t) {
    if constexpr (G == 2) return ((t + 1) >> 1) - 1;
    else return t - 1;
}
// Source groups a target row receives from, per axis.
template <int G> struct GroupSlots { static constexpr int value = G == 1 ? 3 : 2; };

// One source row (ys, zs) of the wave's group: row JY, layer KZ of the group.
// Its contributions go to the accumulators [KZ + 0..2][JY + 0..2] (A = G + 2
// target rows per axis).
// Waves per SIMD asked of the compiler.  The Kahan source (2 x 2 groups) would take
// 170 registers per lane, two waves; in 168, three waves, with two words kept in
// memory from the prologue to the final stores: 400 -> 318 us for the bed of 10
// million, 88 -> 67 for 100,000 particles in 4.2 million cells.
template <typename T, int SM, int MODE> struct RowWaves {
    static constexpr int value = std::is_same<T, float>::value && SM == kSumKahan && MODE == kForce ? 3 : 1;
};

template <typename T, int SM, int MODE, int JY, int KZ, int A>
__device__ __forceinline__ void deposit_source_row(RowSum<T, SM> (&acc)[A][A][DepNc<MODE>::value],
                                                   RowStage<T, MODE> &st, int w, int lane, int x0, int ys, int zs,
                                                   const int32_t *__restrict__ start, const vec4<T> *__restrict__ pk,
                                                   vec4<T> *__restrict__ sp, const int32_t *__restrict__ perm,
                                                   const T *__restrict__ drag, int64_t n, const Geo<T> &g) {
    constexpr int NC = DepNc<MODE>::value;
    using W = typename RowSum<T, SM>::W;
    const int nbx = g.nb[0], nby = g.nb[1], nbz = g.nb[2];
    const int x = x0 + lane;
    const int64_t srow = ((int64_t)zs * nby + ys) * nbx;
    const int xa = x0 > 0 ? x0 - 1 : 0;
    const int xb = (x0 + kWave < nbx ? x0 + kWave : nbx - 1);
    const int32_t rs = seg_clamp(start[srow + xa], n), re = seg_clamp(start[srow + xb + 1], n);
    int32_t os = 0, oe = 0;   // the segment's own particles (its neighbours' waves store theirs)
    if constexpr (MODE == kPhi) {
        os = seg_clamp(start[srow + x0], n);
        oe = seg_clamp(start[srow + (x0 + kWave < nbx ? x0 + kWave : nbx)], n);
    }
    int32_t ls = 0, le = 0;
    if (x < nbx) {
        ls = seg_clamp(start[srow + (x > 0 ? x - 1 : 0)], n);
        le = seg_clamp(start[srow + (x < nbx - 1 ? x + 1 : nbx - 1) + 1], n);
    }
    for (int32_t cs = rs; cs < re; cs += kChunk) {       // wave-uniform loop
        const int32_t m = ((cs + kChunk < re) ? cs + kChunk : re) - cs;
        const int32_t ce = cs + m;
        // Staging: every load of the chunk is issued before any is used, so the
        // random-access gathers through perm cost one round trip per chunk
        // rather than one per 64 particles.
        constexpr int KS = kChunk / kWave;
        vec4<T> q[KS];
        int64_t id[KS];
#pragma unroll
        for (int u = 0; u < KS; ++u) {
            const int k = lane + u * kWave;
            id[u] = 0;
            if (k < m) {
                if constexpr (MODE != kPhi) q[u] = sp[cs + k];
                const int64_t i = perm[cs + k];
                id[u] = (i < 0 || i >= n) ? 0 : i;   // perm is a permutation of [0, n)
            }
        }
        T val[KS][NC];
#pragma unroll
        for (int u = 0; u < KS; ++u) {
            if (lane + u * kWave < m) {
                if constexpr (MODE == kPhi) q[u] = pk[id[u]];
                load_values<T, MODE>(id[u], q[u], drag, pk, g.inv_vb, val[u]);
            }
        }
#pragma unroll
        for (int u = 0; u < KS; ++u) {
            const int k = lane + u * kWave;
            if (k < m) {
                const Axis<T> ax = cic_axis(q[u].x, g.sb[0], nbx);
                const Axis<T> ay = cic_axis(q[u].y, g.sb[1], nby);
                const Axis<T> az = cic_axis(q[u].z, g.sb[2], nbz);
                T wy[3], wz[3];
                row_weights(ay, ys, wy);
                row_weights(az, zs, wz);
                vec4<T> r;
                r.x = wy[0];
                r.y = wy[1];
                r.z = wy[2];
                r.w = ax.t;
                st.wy[w][k] = r;
                r.x = wz[0];
                r.y = wz[1];
                r.z = wz[2];
                r.w = as_value(ax.lo | (ax.hi << 16), T(0));
                st.wz[w][k] = r;
                if constexpr (MODE == kPhi) {
                    st.val[w][k] = val[u][0];
                    if (cs + k >= os && cs + k < oe) sp[cs + k] = q[u];
                } else {
                    r.x = val[u][0];
                    r.y = val[u][1];
                    r.z = val[u][2];
                    r.w = NC > 3 ? val[u][NC - 1] : T(0);
                    st.val[w][k] = r;
                }
            }
        }
        wave_sync();
        const int32_t b0 = (ls > cs ? ls : cs) - cs, b1 = (le < ce ? le : ce) - cs;
        // Branch-free: the lanes of a wave hold different particles, so a skip
        // of the zero weights (5 of the 9 target rows, a third of the x
        // visits) would diverge and save nothing; their terms add zeros.
        for (int32_t k = b0; k < b1; ++k) {
            const vec4<T> ry = st.wy[w][k], rz = st.wz[w][k];
            const int nd = as_bits(rz.w);
            const T t = ry.w;
            T wx = T(0);
            if ((nd & 0xffff) == x) wx += T(1) - t;
            if ((nd >> 16) == x) wx += t;
            W v[NC];
            if constexpr (MODE == kPhi) {
                v[0] = W(wx) * W(st.val[w][k]);
            } else {
                const vec4<T> rv = st.val[w][k];
                v[0] = W(wx) * W(rv.x);
                v[1] = W(wx) * W(rv.y);
                v[2] = W(wx) * W(rv.z);
                if constexpr (NC > 3) v[NC - 1] = W(wx) * W(rv.w);
            }
            const W wy[3] = {W(ry.x), W(ry.y), W(ry.z)}, wz[3] = {W(rz.x), W(rz.y), W(rz.z)};
#pragma unroll
            for (int kz = 0; kz < 3; ++kz) {
#pragma unroll
                for (int jy = 0; jy < 3; ++jy) {
                    const W wyz = wy[jy] * wz[kz];
#pragma unroll
                    for (int c = 0; c < NC; ++c) acc[KZ + kz][JY + jy][c].add(wyz, v[c]);
                }
            }
        }
        wave_sync();
    }
}

template <typename T, int SM, int MODE, int GS>
__global__ __launch_bounds__(kBlock, (RowWaves<T, SM, MODE>::value)) void k_deposit_rows(
    const int32_t *__restrict__ start, const vec4<T> *__restrict__ pk, vec4<T> *__restrict__ sp,
    const int32_t *__restrict__ perm, const T *__restrict__ drag, int64_t n, Geo<T> g, T *__restrict__ partial) {
    constexpr int NC = DepNc<MODE>::value, A = GS + 2, S = GroupSlots<GS>::value;
    __shared__ RowStage<T, MODE> st;
    const int w = threadIdx.x / kWave, lane = threadIdx.x % kWave;
    const int nbx = g.nb[0], nby = g.nb[1], nbz = g.nb[2];
    const int nseg = (nbx + kWave - 1) / kWave;
    const int ngy = (nby + GS - 1) / GS, ngz = (nbz + GS - 1) / GS;
    const int64_t nwave = (int64_t)ngy * ngz * nseg;
    const int64_t tile = xcd_tile(blockIdx.x, gridDim.x);
    const int64_t gw = tile * kWavesPerBlock + w;        // (source group, segment)
    if (gw >= nwave) return;                             // wave-uniform; no block barriers below
    const uint32_t grp = (uint32_t)gw / (uint32_t)nseg;   // fewer than 2^31 waves
    const int x0 = (int)((uint32_t)gw - grp * (uint32_t)nseg) * kWave;
    const int gz = (int)(grp / (uint32_t)ngy), gy = (int)(grp - (uint32_t)gz * (uint32_t)ngy);
    const int x = x0 + lane;
    const int y0 = GS * gy, z0 = GS * gz;
    RowSum<T, SM> acc[A][A][NC];   // [target z - (z0 - 1)][target y - (y0 - 1)][component]
    deposit_source_row<T, SM, MODE, 0, 0, A>(acc, st, w, lane, x0, y0, z0, start, pk, sp, perm, drag, n, g);
    if constexpr (GS == 2) {
        if (y0 + 1 < nby)
            deposit_source_row<T, SM, MODE, 1, 0, A>(acc, st, w, lane, x0, y0 + 1, z0, start, pk, sp, perm, drag, n,
                                                     g);
        if (z0 + 1 < nbz) {
            deposit_source_row<T, SM, MODE, 0, 1, A>(acc, st, w, lane, x0, y0, z0 + 1, start, pk, sp, perm, drag, n,
                                                     g);
            if (y0 + 1 < nby)
                deposit_source_row<T, SM, MODE, 1, 1, A>(acc, st, w, lane, x0, y0 + 1, z0 + 1, start, pk, sp, perm, drag,
                                                         n, g);
        }
    }
    if (x >= nbx) return;
#pragma unroll
    for (int kz = 0; kz < A; ++kz) {
        const int tz = z0 - 1 + kz;
        if (tz < 0 || tz >= nbz) continue;
        const int sz = gz - group_lo<GS>(tz);             // 0 .. S - 1
#pragma unroll
        for (int jy = 0; jy < A; ++jy) {
            const int ty = y0 - 1 + jy;
            if (ty < 0 || ty >= nby) continue;
            const int slot = sz * S + (gy - group_lo<GS>(ty));
            const int64_t tc = ((int64_t)tz * nby + ty) * nbx + x;
#pragma unroll
            for (int c = 0; c < NC; ++c) partial[((int64_t)slot * NC + c) * g.ncell + tc] = T(acc[kz][jy][c].s);
        }
    }
}

template <typename T, int SM, int MODE, int GS>
__global__ __launch_bounds__(kBlock) void k_deposit_sum(const T *__restrict__ partial, Geo<T> g,
                                                        const T *__restrict__ P, const T *__restrict__ Plo,
                                                        T *__restrict__ out, T *__restrict__ out2, T *__restrict__ G,
                                                        double *__restrict__ part, int64_t ps) {
    constexpr int NC = DepNc<MODE>::value, S = GroupSlots<GS>::value;
    __shared__ double red[kWavesPerBlock];
    const int64_t c = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    double v[4] = {0.0, 0.0, 0.0, 0.0};
    if (c < g.ncell) {
        int cx, cy, cz;
        decode_cell(c, g.nb, cx, cy, cz);
        CellSum<T, SM> acc[NC];
        const int gzl = group_lo<GS>(cz), gyl = group_lo<GS>(cy);
        const int ngy = (g.nb[1] + GS - 1) / GS, ngz = (g.nb[2] + GS - 1) / GS;
        GradLoads<T> gl;
        if constexpr (MODE == kForce) gl = load_gradient(c, cx, cy, cz, g, P, Plo);
        // all S x S slots loaded at once (in the partial buffer whether or not
        // their source group exists), then the existing ones summed in order
        T pv[S * S][NC];
#pragma unroll
        for (int slot = 0; slot < S * S; ++slot)
#pragma unroll
            for (int k = 0; k < NC; ++k) pv[slot][k] = partial[((int64_t)slot * NC + k) * g.ncell + c];
#pragma unroll
        for (int sz = 0; sz < S; ++sz)
#pragma unroll
            for (int sy = 0; sy < S; ++sy) {
                const bool has = gzl + sz >= 0 && gzl + sz < ngz && gyl + sy >= 0 && gyl + sy < ngy;
                if (has)
#pragma unroll
                    for (int k = 0; k < NC; ++k) acc[k].add(pv[sz * S + sy][k]);
            }
        if constexpr (MODE == kForce) {
            const T fx = -acc[0].value() * g.inv_vb, fy = -acc[1].value() * g.inv_vb, fz = -acc[2].value() * g.inv_vb;
            out[c] = fx;
            out[g.ncell + c] = fy;
            out[2 * g.ncell + c] = fz;
            v[0] = fx; v[1] = fy; v[2] = fz;
            write_gradient(gl, c, cx, cy, cz, g, G);
        } else if constexpr (MODE == kSemi) {
            out[c] = acc[0].value() * g.inv_vb;
            for (int k = 0; k < 3; ++k) out2[k * g.ncell + c] = acc[k + 1].value() * g.inv_vb;
            for (int k = 0; k < 4; ++k) v[k] = (double)(acc[k].value() * g.inv_vb);
        } else {
            out[c] = acc[0].value();
            v[0] = (double)acc[0].value();
        }
    }
    if constexpr (MODE == kPhi) {
        const double t = block_sum(v[0], red);
        const double m = block_max(v[0], red);
        if (threadIdx.x == 0) {
            part[SL_PHISUM * ps + blockIdx.x] = t;
            part[SL_MAXPHI * ps + blockIdx.x] = m;
        }
    } else if constexpr (MODE == kForce) {
        for (int k = 0; k < 3; ++k) {
            const double t = block_sum(v[k], red);
            if (threadIdx.x == 0) part[(SL_FB + k) * ps + blockIdx.x] = t;
        }
    } else {
        const int slots[4] = {SL_KB, SL_KUB, SL_KUB + 1, SL_KUB + 2};
        for (int k = 0; k < 4; ++k) {
            const double t = block_sum(v[k], red);
            if (threadIdx.x == 0) part[slots[k] * ps + blockIdx.x] = t;
        }
    }
}

// ---------------------------------------------------------------------------
// Host side
// ---------------------------------------------------------------------------
int deposit_blocks(int64_t n, int64_t ncell, int cic) {
    if (cic) return (int)((ncell + kBlock - 1) / kBlock);   // pass 2
    const int cells = ngp_cells(n, ncell);   // NGP: each loops over its groups of cells
    return (int)std::min((ncell + cells - 1) / cells, most_partials(n, ncell));
}

static int64_t row_waves(const int nb[3], int G) {
    const int64_t nseg = (nb[0] + kWave - 1) / kWave;
    return (int64_t)((nb[1] + G - 1) / G) * ((nb[2] + G - 1) / G) * nseg;
}

// Source rows per group of the CIC row pass: 2 x 2 (each target row receives 4
// partials) unless that leaves fewer than 4096 waves (four per SIMD of the
// chip), then single rows (9 partials per target, four times the waves).
int deposit_group(const int nb[3]) { return row_waves(nb, 2) < 4096 ? 1 : 2; }

static int row_blocks(const int nb[3], int G) {
    return (int)((row_waves(nb, G) + kWavesPerBlock - 1) / kWavesPerBlock);
}

template <typename T, int SM, int MODE>
static int launch_deposit(const StepArgs<T> &a, T *out, T *out2, hipStream_t st, const char *sum_mark) {
    const int nblk = deposit_blocks(a.n, a.g.ncell, a.cic);
    // the packed particles until the velocity is sampled; (beta, beta u_p) once the drag has run
    const vec4<T> *pk = a.uf4;
    if (a.cic) {
        auto rows_and_sums = [&](auto gc) {
            constexpr int GS = decltype(gc)::value;
            hipLaunchKernelGGL((k_deposit_rows<T, SM, MODE, GS>), dim3(row_blocks(a.g.nb, GS)), dim3(kBlock), 0, st,
                               a.start, pk, a.sp, a.perm, a.drag, a.n, a.g, a.dep_partial);
            a.mk->mark(sum_mark, st);
            hipLaunchKernelGGL((k_deposit_sum<T, SM, MODE, GS>), dim3(nblk), dim3(kBlock), 0, st, a.dep_partial, a.g,
                               a.P, a.Plo, out, out2, a.G, a.part, a.part_stride);
        };
        if (deposit_group(a.g.nb) == 1) rows_and_sums(std::integral_constant<int, 1>{});
        else rows_and_sums(std::integral_constant<int, 2>{});
    } else {
        const int cells = ngp_cells(a.n, a.g.ncell);
        auto groups = [&](auto wide) {
            hipLaunchKernelGGL((k_deposit_ngp<T, SM, MODE, decltype(wide)::value>), dim3(nblk), dim3(kBlock), 0, st,
                               a.start, pk, a.sp, a.perm, a.drag, a.n, a.g, a.P, a.Plo, out, out2, a.G, a.part,
                               a.part_stride, cells);
        };
        if (cells == kBlock) groups(std::true_type{});
        else groups(std::false_type{});
    }
    return nblk;
}

template <typename T, int SM> int launch_deposit_phi(const StepArgs<T> &a, hipStream_t st) {
    return launch_deposit<T, SM, kPhi>(a, a.phi, nullptr, st, "deposit_phi_sum");
}

template <typename T, int SM> int launch_deposit_force(const StepArgs<T> &a, hipStream_t st) {
    return launch_deposit<T, SM, kForce>(a, a.F, nullptr, st, "deposit_force_sum");
}

template <typename T, int SM> int launch_deposit_semi(const StepArgs<T> &a, hipStream_t st) {
    return launch_deposit<T, SM, kSemi>(a, a.K, a.KU, st, "deposit_semi_sum");
}

template int launch_deposit_phi<float, kSumPlain>(const StepArgs<float> &, hipStream_t);
template int launch_deposit_phi<float, kSumKahan>(const StepArgs<float> &, hipStream_t);
template int launch_deposit_phi<float, kSumWide>(const StepArgs<float> &, hipStream_t);
template int launch_deposit_phi<double, kSumPlain>(const StepArgs<double> &, hipStream_t);
template int launch_deposit_force<float, kSumPlain>(const StepArgs<float> &, hipStream_t);
template int launch_deposit_force<float, kSumKahan>(const StepArgs<float> &, hipStream_t);
template int launch_deposit_force<float, kSumWide>(const StepArgs<float> &, hipStream_t);
template int launch_deposit_force<double, kSumPlain>(const StepArgs<double> &, hipStream_t);
template int launch_deposit_semi<float, kSumPlain>(const StepArgs<float> &, hipStream_t);
template int launch_deposit_semi<float, kSumKahan>(const StepArgs<float> &, hipStream_t);
template int launch_deposit_semi<float, kSumWide>(const StepArgs<float> &, hipStream_t);
template int launch_deposit_semi<double, kSumPlain>(const StepArgs<double> &, hipStream_t);

}  // namespace cpl
