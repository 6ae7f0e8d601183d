// sort.hip -- binning of particles into bulk cells and the deterministic,
// stable LSD radix sort that yields the canonical (cell, id) order.
//
// The particle -> cell connectivity changes with every coupling step because
// the particles move (Sec. 2.2); it is rebuilt here from scratch each step:
//
//   k_bin          containing cell per particle (output `cell`), the packed
//                  input-order copy pk = (x, y, z, d) with the position clamped
//                  into the box, and the digit histogram of the first radix
//                  pass, per tile;
//   k_radix_hist   digit histogram per tile for later passes;
//   k_radix_prefix exclusive prefix over tiles of every digit, digit totals;
//   k_radix_scatter stable ranking inside a tile (wave ballots, LDS staging) and
//                  coalesced scatter to the digit's output run;
//   k_count_scatter  instead of all that follows k_bin, for few particles in few
//                  cells: one pass with the whole cell index as the digit;
//   k_segment_starts  start[c] = first sorted position with cell >= c, set by
//                  the sorted positions where the key changes (long runs of
//                  empty cells are left to the next kernel);
//   k_segment_counts  the starts left unset (binary search of the sorted keys)
//                  and count[c] = start[c+1] - start[c].
//
// Keys are cell indices < ncell; ids are the input order, so a stable LSD sort
// starting from the identity order gives ascending (cell, id).  Integer atomics
// are used only on LDS histogram bins (exact counts); no float atomics anywhere.
#include <algorithm>
#include <type_traits>

#include "common.hpp"
#include "launch.hpp"

namespace cpl {

constexpr int kMaxItems = 16;                      // most keys per thread of a tile (the kernels' ITEMS)
constexpr int kMaxDigits = 256;                    // radix <= 8 bits per pass

// A start entry not yet known: k_bin marks every entry so, k_segment_starts sets
// all but those inside long runs of empty cells, k_segment_counts the rest.
constexpr int32_t kUnset = -1;

// Workgroups [0, ntile) bin the particles of their tile of kBlock x ITEMS; every
// workgroup of the grid (which may be larger, to cover the cells) also marks a
// share of start[0 .. nstart) unset.  The particles are taken kBinBatch per
// thread at a time, all their loads issued before the first is used.
// COUNT: the histogram is that of the counting sort, 16-bit counts of all cells
// tile by tile (rows of ndig, a multiple of 8).
constexpr int kBinBatch = 4;
constexpr int64_t kCountCells = 8192;   // most cells of a counting sort (multiple of 8)
template <typename T, int ITEMS, bool COUNT>
__global__ __launch_bounds__(kBlock) void k_bin(const T *__restrict__ pos, const T *__restrict__ diam, int64_t n,
                                                Geo<T> g, int32_t *__restrict__ cell, vec4<T> *__restrict__ pk,
                                                uint32_t *__restrict__ hist,
                                                int ntile, int ndig, double *__restrict__ part_nout,
                                                int32_t *__restrict__ start, int64_t nstart) {
    __shared__ uint32_t h[COUNT ? kCountCells : kMaxDigits];
    __shared__ double red[kWavesPerBlock];
    for (int64_t c = (int64_t)blockIdx.x * kBlock + threadIdx.x; c < nstart; c += (int64_t)gridDim.x * kBlock)
        start[c] = kUnset;
    if ((int)blockIdx.x >= ntile) return;   // uniform over the workgroup, before any barrier
    for (int d = threadIdx.x; d < ndig; d += kBlock) h[d] = 0;
    __syncthreads();
    const int64_t base = (int64_t)blockIdx.x * kBlock * ITEMS + threadIdx.x;
    double nout = 0.0;
    constexpr int NB = ITEMS < kBinBatch ? ITEMS : kBinBatch;
    for (int it0 = 0; it0 < ITEMS; it0 += NB) {
        T xs[NB][3], ds[NB];
#pragma unroll
        for (int u = 0; u < NB; ++u) {
            int64_t p = base + (int64_t)(it0 + u) * kBlock;
            p = p < n ? p : n - 1;
#pragma unroll
            for (int k = 0; k < 3; ++k) xs[u][k] = pos[3 * p + k];
            ds[u] = diam[p];
        }
#pragma unroll
        for (int u = 0; u < NB; ++u) {
            const int64_t p = base + (int64_t)(it0 + u) * kBlock;
            if (p >= n) continue;
            int outside = 0;
            const T x = clamp_coord(xs[u][0], g.L[0], outside);
            const T y = clamp_coord(xs[u][1], g.L[1], outside);
            const T z = clamp_coord(xs[u][2], g.L[2], outside);
            const int ix = cell_axis(x, g.sb[0], g.nb[0]);
            const int iy = cell_axis(y, g.sb[1], g.nb[1]);
            const int iz = cell_axis(z, g.sb[2], g.nb[2]);
            const int32_t c = ix + g.nb[0] * (iy + g.nb[1] * iz);
            cell[p] = c;
            vec4<T> q;
            q.x = x;
            q.y = y;
            q.z = z;
            q.w = ds[u];
            pk[p] = q;
            const uint32_t d = COUNT ? min((uint32_t)c, (uint32_t)ndig - 1u) : (uint32_t)c & (ndig - 1);   // in bounds
            atomicAdd(&h[d], 1u);
            nout += outside;
        }
    }
    __syncthreads();
    if constexpr (COUNT) {
        for (int d = threadIdx.x; d < ndig / 2; d += kBlock)
            hist[(int64_t)blockIdx.x * (ndig / 2) + d] = h[2 * d] | h[2 * d + 1] << 16;
    } else {
        for (int d = threadIdx.x; d < ndig; d += kBlock) hist[(int64_t)d * ntile + blockIdx.x] = h[d];
    }
    double t = block_sum(nout, red);
    if (threadIdx.x == 0) part_nout[blockIdx.x] = t;
}

template <int ITEMS>
__global__ __launch_bounds__(kBlock) void k_radix_hist(const uint32_t *__restrict__ keys, int64_t n, int shift,
                                                       int bits, uint32_t *__restrict__ hist, int ntile) {
    __shared__ uint32_t h[kMaxDigits];
    const int ndig = 1 << bits;
    for (int d = threadIdx.x; d < ndig; d += kBlock) h[d] = 0;
    __syncthreads();
    const int64_t base = (int64_t)blockIdx.x * kBlock * ITEMS + threadIdx.x;
    uint32_t k[ITEMS];
#pragma unroll
    for (int it = 0; it < ITEMS; ++it) {
        const int64_t p = base + (int64_t)it * kBlock;
        k[it] = keys[p < n ? p : n - 1];
    }
#pragma unroll
    for (int it = 0; it < ITEMS; ++it)
        if (base + (int64_t)it * kBlock < n) atomicAdd(&h[(k[it] >> shift) & (ndig - 1)], 1u);
    __syncthreads();
    for (int d = threadIdx.x; d < ndig; d += kBlock) hist[(int64_t)d * ntile + blockIdx.x] = h[d];
}

// One workgroup per digit: exclusive prefix over the tiles (in place) and the
// digit's total.  Each thread takes a contiguous run of tiles: its sum, one
// scan over the workgroup, then the run's prefixes (two barriers whatever the
// number of tiles).
__global__ __launch_bounds__(kBlock) void k_radix_prefix(uint32_t *__restrict__ hist, int ntile,
                                                         uint32_t *__restrict__ totals) {
    __shared__ uint32_t wsum[kWavesPerBlock];
    uint32_t *row = hist + (int64_t)blockIdx.x * ntile;
    const int lane = threadIdx.x % kWave, w = threadIdx.x / kWave;
    const int per = (ntile + kBlock - 1) / kBlock;
    const int i0 = (int)threadIdx.x * per, i1 = i0 + per < ntile ? i0 + per : ntile;
    uint32_t v = 0;
    for (int i = i0; i < i1; ++i) v += row[i];
    uint32_t s = v;   // inclusive wave scan
    for (int o = 1; o < kWave; o <<= 1) {
        const uint32_t u = __shfl_up(s, o, kWave);
        if (lane >= o) s += u;
    }
    if (lane == kWave - 1) wsum[w] = s;
    __syncthreads();
    uint32_t off = s - v;
    for (int k = 0; k < w; ++k) off += wsum[k];
    if (threadIdx.x == kBlock - 1) totals[blockIdx.x] = off + v;
    for (int i = i0; i < i1; ++i) {
        const uint32_t c = row[i];
        row[i] = off;
        off += c;
    }
}

// Stable tile ranking and scatter.  FIRST: values are the input positions (ids).
// Every key and value of a thread is loaded before the first is ranked: the
// ranking is a serial chain through the LDS counters, and a load inside it
// would add a memory round trip per key (10,000 keys: 13.4 us with the loads
// in the chain).  The digits' totals and prefixes are loaded with them, and their
// scan is one with the tile's (after the ranking and apart: a step of 333,337
// particles 133.7 instead of 131.8 us, of 10 million 2966 instead of 2958).
// Digits of 9 bits, two passes for 18-bit keys instead of three, leave runs of two
// to four keys per tile: 24 us a pass instead of 13 for 2 million keys.
template <bool FIRST, int ITEMS>
__global__ __launch_bounds__(kBlock) void k_radix_scatter(const uint32_t *__restrict__ keys_in,
                                                          const uint32_t *__restrict__ vals_in, int64_t n,
                                                          int shift, int bits, const uint32_t *__restrict__ hist,
                                                          const uint32_t *__restrict__ totals, int ntile,
                                                          uint32_t *__restrict__ keys_out,
                                                          uint32_t *__restrict__ vals_out) {
    constexpr int kTile = kBlock * ITEMS, kWaveSpan = kWave * ITEMS;   // keys of a workgroup, of a wave
    __shared__ uint32_t digit_base[kMaxDigits];       // global start of each digit's run
    __shared__ uint32_t local_start[kMaxDigits];      // start of each digit inside the tile
    __shared__ uint32_t wave_cnt[kWavesPerBlock][kMaxDigits];
    __shared__ uint32_t skey[kTile];
    __shared__ uint32_t sval[kTile];
    __shared__ uint32_t scan_tmp[2][kWavesPerBlock];

    const int ndig = 1 << bits;
    const uint32_t dmask = ndig - 1;
    const int lane = threadIdx.x % kWave, w = threadIdx.x / kWave;
    const int64_t tile0 = (int64_t)blockIdx.x * kTile;
    const int tile_n = (int)((n - tile0) < kTile ? (n - tile0) : kTile);

    for (int d = threadIdx.x; d < kMaxDigits; d += kBlock) {
        wave_cnt[0][d] = wave_cnt[1][d] = wave_cnt[2][d] = wave_cnt[3][d] = 0;
    }
    __syncthreads();

    // ---- rank: wave w owns keys [w*kWaveSpan, (w+1)*kWaveSpan) of the tile ----
    uint32_t key[ITEMS], val[ITEMS], rank[ITEMS];
    const uint64_t lt_mask = (lane == 0) ? 0ull : (~0ull >> (kWave - lane));
#pragma unroll
    for (int it = 0; it < ITEMS; ++it) {
        int li = w * kWaveSpan + it * kWave + lane;   // position inside the tile
        li = li < tile_n ? li : tile_n - 1;
        key[it] = keys_in[tile0 + li];
        val[it] = FIRST ? (uint32_t)(tile0 + li) : vals_in[tile0 + li];
    }
    static_assert(kMaxDigits == kBlock, "a digit per thread");
    const int dt = (int)threadIdx.x < ndig ? (int)threadIdx.x : 0;
    uint32_t g = totals[dt], hb = hist[(int64_t)dt * ntile + blockIdx.x];
    if ((int)threadIdx.x >= ndig) g = 0;
#pragma unroll
    for (int it = 0; it < ITEMS; ++it) {
        const bool valid = w * kWaveSpan + it * kWave + lane < tile_n;
        const uint32_t d = (key[it] >> shift) & dmask;
        uint64_t peers = __ballot(valid);
        for (int b = 0; b < bits; ++b) {
            bool bit = (d >> b) & 1u;
            uint64_t m = __ballot(bit);
            peers &= bit ? m : ~m;
        }
        uint32_t before = __popcll(peers & lt_mask);
        uint32_t cnt = valid ? wave_cnt[w][d] : 0u;
        // the lowest lane of each peer group advances the running count
        bool leader = valid && ((peers & lt_mask) == 0ull);
        __builtin_amdgcn_wave_barrier();
        if (leader) wave_cnt[w][d] = cnt + (uint32_t)__popcll(peers);
        __builtin_amdgcn_wave_barrier();
        rank[it] = valid ? cnt + before : 0xffffffffu;
    }
    __syncthreads();

    // ---- per digit (one per thread): prefix over waves; exclusive scans over the
    // digits of the tile's counts and of the global totals ---------------------
    uint32_t tot = 0;
    for (int q = 0; q < kWavesPerBlock; ++q) {
        const uint32_t c = wave_cnt[q][threadIdx.x];
        wave_cnt[q][threadIdx.x] = tot;
        tot += c;
    }
    uint32_t s = tot, gs = g;
    for (int o = 1; o < kWave; o <<= 1) {
        const uint32_t u = __shfl_up(s, o, kWave), gu = __shfl_up(gs, o, kWave);
        if (lane >= o) {
            s += u;
            gs += gu;
        }
    }
    if (lane == kWave - 1) {
        scan_tmp[0][w] = s;
        scan_tmp[1][w] = gs;
    }
    __syncthreads();
    uint32_t off = s - tot, goff = gs - g;
    for (int q = 0; q < w; ++q) {
        off += scan_tmp[0][q];
        goff += scan_tmp[1][q];
    }
    local_start[threadIdx.x] = off;
    digit_base[threadIdx.x] = goff + hb;
    __syncthreads();

    // ---- stage the tile in digit order in LDS --------------------------------
#pragma unroll
    for (int it = 0; it < ITEMS; ++it) {
        if (rank[it] != 0xffffffffu) {
            uint32_t d = (key[it] >> shift) & dmask;
            uint32_t lp = local_start[d] + wave_cnt[w][d] + rank[it];
            skey[lp] = key[it];
            sval[lp] = val[it];
        }
    }
    __syncthreads();

    // ---- write out: consecutive threads write consecutive positions of a run --
    for (int i = threadIdx.x; i < tile_n; i += kBlock) {
        uint32_t k = skey[i];
        uint32_t d = (k >> shift) & dmask;
        uint32_t dst = digit_base[d] + (i - local_start[d]);
        if (dst < (uint64_t)n) {   // always true for a consistent histogram; guards the store
            keys_out[dst] = k;
            vals_out[dst] = sval[i];
        }
    }
}

// The counting sort: one pass whose digit is the cell index.  Workgroup b forms,
// from the 16-bit counts of every tile (rows of ndig, a multiple of 8, at most
// kCountCells), the first sorted position of each cell and its own tile's place in
// it, ranks its tile as k_radix_scatter does and writes it out; the workgroups
// share the writing of start and count.  There are fewer than 2^16 particles, so
// two counts are summed in a 32-bit word without a carry.  It takes the place of
// seven launches (two radix passes, the segments), each of which lasts a few
// memory round trips: 6.6 us instead of 22.5 for 10,000 particles in 512 cells,
// 10.9 instead of 25.8 for 20,011 in 4199 (the tiles' counts, one batch of
// kCountRows loads after the other, are the longest of its chains).
constexpr int64_t kCountKeys = 65535;
constexpr int kCountItems = 4, kCountRows = 16;           // keys per thread of the ranking waves, tile rows in flight
constexpr int kCountThreads = (int)(kCountCells / 8);     // a thread sums the counts of eight cells (16 bytes)
static_assert(kCountThreads <= 1024 && kCountThreads >= kBlock, "threads of k_count_scatter");
__global__ __launch_bounds__(kCountThreads) void k_count_scatter(
    const uint32_t *__restrict__ keys_in, int64_t n, int bits, const uint4 *__restrict__ hist, int ntile, int ndig,
    int64_t ncell, uint32_t *__restrict__ keys_out, uint32_t *__restrict__ vals_out, int32_t *__restrict__ start,
    int32_t *__restrict__ count) {
    constexpr int kTile = kBlock * kCountItems, kWaveSpan = kWave * kCountItems, kWaves = kCountThreads / kWave;
    __shared__ __align__(16) uint16_t wave_cnt[kWavesPerBlock][kCountCells];   // keys of each cell, per ranking wave
    __shared__ __align__(16) uint16_t cell_base[kCountCells];                  // first output position in each cell
    __shared__ uint32_t wsum[kWaves];
    const int lane = threadIdx.x % kWave, w = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave), nchunk = ndig / 8;
    const int64_t tile0 = (int64_t)blockIdx.x * kTile;
    const int tile_n = (int)((n - tile0) < kTile ? (n - tile0) : kTile);
    const bool ranks = w < kWavesPerBlock;   // the first four waves rank the tile

    uint32_t key[kCountItems];
#pragma unroll
    for (int it = 0; it < kCountItems; ++it) {
        const int li = w * kWaveSpan + it * kWave + lane;
        key[it] = keys_in[tile0 + (li < tile_n ? li : tile_n - 1)];
    }
    const int c = threadIdx.x;
    if (c < nchunk)
        for (int q = 0; q < kWavesPerBlock; ++q) reinterpret_cast<uint4 *>(wave_cnt[q])[c] = make_uint4(0u, 0u, 0u, 0u);

    // the thread's eight cells: counts in all tiles (tot) and in those before this
    // one (bef), two to a word
    uint32_t tot[4] = {0, 0, 0, 0}, bef[4] = {0, 0, 0, 0}, sum = 0;
    if (w * kWave < nchunk) {
        const uint4 *row = hist + (c < nchunk ? c : nchunk - 1);
        for (int t0 = 0; t0 < ntile; t0 += kCountRows) {
            uint4 v[kCountRows];
#pragma unroll
            for (int u = 0; u < kCountRows; ++u) v[u] = row[(int64_t)(t0 + u < ntile ? t0 + u : ntile - 1) * nchunk];
#pragma unroll
            for (int u = 0; u < kCountRows; ++u) {
                const uint32_t in = t0 + u < ntile ? ~0u : 0u, lt = t0 + u < (int)blockIdx.x ? ~0u : 0u;
                const uint32_t x[4] = {v[u].x, v[u].y, v[u].z, v[u].w};
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    tot[e] += x[e] & in;
                    bef[e] += x[e] & lt;
                }
            }
        }
#pragma unroll
        for (int e = 0; e < 4; ++e) sum += (tot[e] & 0xffffu) + (tot[e] >> 16);
        if (c >= nchunk) sum = 0;
    }
    uint32_t scan = sum;   // inclusive wave scan
    for (int o = 1; o < kWave; o <<= 1) {
        const uint32_t u = __shfl_up(scan, o, kWave);
        if (lane >= o) scan += u;
    }
    if (lane == kWave - 1) wsum[w] = scan;
    __syncthreads();
    if (c < nchunk) {
        uint32_t pos = scan - sum;
        for (int q = 0; q < w; ++q) pos += wsum[q];
        const bool mine = c % ntile == (int)blockIdx.x;
        uint32_t out[4] = {0, 0, 0, 0};
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const int sh = 16 * (e & 1);
            const uint32_t b = (bef[e / 2] >> sh) & 0xffffu, m = (tot[e / 2] >> sh) & 0xffffu;
            out[e / 2] |= (pos + b) << sh;
            if (mine && 8 * c + e < ncell) {
                start[8 * c + e] = (int32_t)pos;
                count[8 * c + e] = (int32_t)m;
            }
            pos += m;
        }
        reinterpret_cast<uint4 *>(cell_base)[c] = make_uint4(out[0], out[1], out[2], out[3]);
    }
    if (blockIdx.x == 0 && threadIdx.x == 0) start[ncell] = (int32_t)n;

    // rank: wave w owns keys [w*kWaveSpan, (w+1)*kWaveSpan) of the tile
    uint32_t rank[kCountItems];
    if (ranks) {
        const uint64_t lt_mask = (lane == 0) ? 0ull : (~0ull >> (kWave - lane));
#pragma unroll
        for (int it = 0; it < kCountItems; ++it) {
            const bool valid = w * kWaveSpan + it * kWave + lane < tile_n;
            const uint32_t d = min(key[it], (uint32_t)ndig - 1u);   // always below; keeps LDS in bounds
            uint64_t peers = __ballot(valid);
            for (int b = 0; b < bits; ++b) {
                const bool bit = (d >> b) & 1u;
                const uint64_t m = __ballot(bit);
                peers &= bit ? m : ~m;
            }
            const uint32_t cnt = valid ? wave_cnt[w][d] : 0u;
            const bool leader = valid && ((peers & lt_mask) == 0ull);
            __builtin_amdgcn_wave_barrier();
            if (leader) wave_cnt[w][d] = (uint16_t)(cnt + (uint32_t)__popcll(peers));
            __builtin_amdgcn_wave_barrier();
            rank[it] = cnt + __popcll(peers & lt_mask);
        }
    }
    __syncthreads();
    if (!ranks) return;
#pragma unroll
    for (int it = 0; it < kCountItems; ++it) {
        const int li = w * kWaveSpan + it * kWave + lane;
        const uint32_t d = min(key[it], (uint32_t)ndig - 1u);
        uint32_t dst = cell_base[d] + rank[it];
#pragma unroll
        for (int q = 0; q < kWavesPerBlock - 1; ++q) dst += q < w ? wave_cnt[q][d] : 0;
        if (li < tile_n && dst < (uint64_t)n) {
            keys_out[dst] = key[it];
            vals_out[dst] = (uint32_t)(tile0 + li);
        }
    }
}

// start[c] = first sorted position with key >= c, for c in [0, ncell].  Every
// sorted position i whose key differs from its predecessor's (with key[-1] = -1
// and key[n] = ncell) sets start[c] = i for the cells c in (key[i-1], key[i]],
// so every entry is written at most once and the keys are read once, coalesced,
// without searches.  A gap of more than kGapLane cells (a run of empty cells)
// is filled by the whole wave together; one of more than kGapWave cells is left
// unset for k_segment_counts, which spreads it over the grid (a single wave
// filling millions of empty cells would serialise the step).
constexpr int kGapLane = 32;
constexpr int64_t kGapWave = 4096;

__global__ __launch_bounds__(kBlock) void k_segment_starts(const uint32_t *__restrict__ skeys, int64_t n,
                                                           int64_t ncell, int32_t *__restrict__ start) {
    const int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x;   // sorted position, 0 .. n
    const int lane = threadIdx.x % kWave;
    int32_t lo = 0, hi = -1;   // the cells set to i
    if (i <= n) {
        // keys are cells < ncell; the clamp only keeps the stores in bounds
        auto key = [&](int64_t k) { const int64_t v = skeys[k]; return (int32_t)(v < ncell ? v : ncell - 1); };
        lo = (i == 0 ? -1 : key(i - 1)) + 1;
        hi = i == n ? (int32_t)ncell : key(i);
    }
    const int32_t len = hi - lo + 1;
    if (len > 0 && len <= kGapLane)
        for (int32_t c = lo; c <= hi; ++c) start[c] = (int32_t)i;
    uint64_t m = __ballot(len > kGapLane);   // wave-uniform
    while (m) {
        const int l = __ffsll((unsigned long long)m) - 1;
        m &= m - 1;
        const int32_t glo = __shfl(lo, l, kWave), ghi = __shfl(hi, l, kWave), gi = __shfl((int32_t)i, l, kWave);
        if ((int64_t)ghi - glo + 1 > kGapWave) continue;   // left unset (wave-uniform)
        for (int64_t c = (int64_t)glo + lane; c <= ghi; c += kWave) start[c] = gi;   // 64-bit: no wrap near 2^31
    }
}

// First sorted position i in [0, n] with key[i] >= c (binary search).
__device__ __forceinline__ int32_t first_at_least(const uint32_t *__restrict__ skeys, int64_t n, int64_t c) {
    int64_t lo = 0, hi = n;
    while (lo < hi) {
        const int64_t mid = (lo + hi) >> 1;
        if ((int64_t)skeys[mid] < c) lo = mid + 1;
        else hi = mid;
    }
    return (int32_t)lo;
}

// Thread c in [0, ncell]: resolves start[c] if it is unset, and count[c] =
// start[c+1] - start[c] (an unset start[c+1] is resolved here too; its own
// thread stores the same value).
__global__ __launch_bounds__(kBlock) void k_segment_counts(int32_t *start, int64_t ncell,
                                                           const uint32_t *__restrict__ skeys, int64_t n,
                                                           int32_t *__restrict__ count) {
    const int64_t c = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (c > ncell) return;
    int32_t v = start[c];
    if (v == kUnset) {
        v = first_at_least(skeys, n, c);
        start[c] = v;
    }
    if (c < ncell) {
        int32_t w = start[c + 1];
        if (w == kUnset) w = first_at_least(skeys, n, c + 1);
        count[c] = w - v;
    }
}

// ---------------------------------------------------------------------------
// Host side
// ---------------------------------------------------------------------------

// Keys per thread of a tile: the fewest that leave at most kTilesWanted tiles.
// A tile's ranking is a serial chain of ITEMS keys per wave, so fewer keys per
// tile shorten a launch that cannot fill the chip (four tiles per compute unit
// fill it); more tiles than that only lengthen the per-digit prefix.
constexpr int64_t kTilesWanted = 1024;
static int64_t tiles_of(int64_t n, int items) { return (n + (int64_t)kBlock * items - 1) / ((int64_t)kBlock * items); }
static int sort_items(int64_t n, int64_t max_tiles) {
    for (int items : {4, 8})
        if (tiles_of(n, items) <= kTilesWanted && tiles_of(n, items) <= max_tiles) return items;
    return kMaxItems;
}

int64_t sort_tiles_min(int64_t n) { return tiles_of(n > 0 ? n : 1, kMaxItems); }
int64_t sort_tiles_max(int64_t n) {
    return std::max(sort_tiles_min(n), std::min(tiles_of(n > 0 ? n : 1, 4), kTilesWanted));
}
int sort_tiles(int64_t n, int64_t max_tiles) { return (int)tiles_of(n, sort_items(n, max_tiles)); }

// The counting sort is taken where its counts fit 16 bits and the workgroup's LDS,
// and the histogram scratch (that of a step over static memory may not).  At the
// limits too it is the faster: a whole step of 65,000 particles takes 54.7 us in
// 4096 cells (75.8 with the radix passes) and 54.9 in 8000 (76.3).
static int count_digits(int64_t ncell) { return (int)((ncell + 7) / 8 * 8); }
size_t count_sort_bytes(int64_t nmax, int64_t ncell) {
    if (ncell > kCountCells || nmax <= 0) return 0;
    return sizeof(uint16_t) * count_digits(ncell) * tiles_of(std::min(nmax, kCountKeys), kCountItems);
}
static bool counts_cells(int64_t n, int64_t ncell, const SortScratch &s) {
    const size_t need = count_sort_bytes(n, ncell);
    return n <= kCountKeys && need > 0 && need <= s.hist_bytes && sort_items(n, s.max_tiles) == kCountItems;
}

void sort_plan(int64_t ncell, int *npass, int widths[4]) {
    int bits = 1;
    while ((int64_t(1) << bits) < ncell) ++bits;
    int p = (bits + 7) / 8;
    int base = bits / p, extra = bits % p;
    for (int i = 0; i < p; ++i) widths[i] = base + (i < extra ? 1 : 0);
    *npass = p;
}

// f(integral_constant) for the tile size of `items` keys per thread.
template <typename F> static void with_items(int items, F f) {
    if (items == 4) f(std::integral_constant<int, 4>{});
    else if (items == 8) f(std::integral_constant<int, 8>{});
    else f(std::integral_constant<int, kMaxItems>{});
}

// One radix pass (its histograms are there already unless `hist`); vin NULL: the
// values are the positions.
static void radix_pass(const uint32_t *kin, const uint32_t *vin, int64_t n, int shift, int bits, bool hist, int items,
                       const SortScratch &s, uint32_t *kout, uint32_t *vout, Marker *mk, hipStream_t st) {
    const int ntile = (int)tiles_of(n, items);
    with_items(items, [&](auto ic) {
        constexpr int I = decltype(ic)::value;
        if (hist) {
            mk->mark("radix_hist", st);
            hipLaunchKernelGGL(k_radix_hist<I>, dim3(ntile), dim3(kBlock), 0, st, kin, n, shift, bits, s.hist, ntile);
        }
        mk->mark("radix_prefix", st);
        hipLaunchKernelGGL(k_radix_prefix, dim3(1 << bits), dim3(kBlock), 0, st, s.hist, ntile, s.totals);
        mk->mark("radix_scatter", st);
        if (vin)
            hipLaunchKernelGGL((k_radix_scatter<false, I>), dim3(ntile), dim3(kBlock), 0, st, kin, vin, n, shift, bits,
                               s.hist, s.totals, ntile, kout, vout);
        else
            hipLaunchKernelGGL((k_radix_scatter<true, I>), dim3(ntile), dim3(kBlock), 0, st, kin, vin, n, shift, bits,
                               s.hist, s.totals, ntile, kout, vout);
    });
}

template <typename T>
hipError_t launch_bin_sort(const T *pos, const T *diam, int64_t n, const Geo<T> &g, int32_t *cell, vec4<T> *pk,
                           int32_t *perm, int32_t *start, int32_t *count, const SortScratch &s, double *part_nout,
                           const uint32_t **sorted_keys, Marker *mk, hipStream_t st) {
    int npass, widths[4];
    sort_plan(g.ncell, &npass, widths);
    const int items = sort_items(n, s.max_tiles);
    const int ntile = n > 0 ? (int)tiles_of(n, items) : 0;
    if (counts_cells(n, g.ncell, s)) {
        const int ndig = count_digits(g.ncell);
        mk->mark("bin", st);
        hipLaunchKernelGGL((k_bin<T, kCountItems, true>), dim3(ntile), dim3(kBlock), 0, st, pos, diam, n, g, cell, pk,
                           s.hist, ntile, ndig, part_nout, start, (int64_t)0);
        int bits = 1;
        while ((1 << bits) < ndig) ++bits;
        mk->mark("count_scatter", st);
        hipLaunchKernelGGL(k_count_scatter, dim3(ntile), dim3(kCountThreads), 0, st, (const uint32_t *)cell, n, bits,
                           (const uint4 *)s.hist, ntile, ndig, g.ncell, s.keys_a, (uint32_t *)perm, start, count);
        *sorted_keys = s.keys_a;
        return hipGetLastError();
    }
    // the binning grid also covers start[0 .. ncell] (marked unset)
    const int64_t nstart = g.ncell + 1;
    const int bin_blocks = (int)std::max<int64_t>(ntile, tiles_of(nstart, kMaxItems));
    mk->mark("bin", st);
    with_items(items, [&](auto ic) {
        hipLaunchKernelGGL((k_bin<T, decltype(ic)::value, false>), dim3(bin_blocks), dim3(kBlock), 0, st, pos, diam, n, g,
                           cell, pk, s.hist, ntile, 1 << widths[0], part_nout, start, nstart);
    });
    *sorted_keys = s.keys_a;
    if (n > 0) {
        int shift = 0;
        const uint32_t *kin = (const uint32_t *)cell;
        const uint32_t *vin = nullptr;
        for (int p = 0; p < npass; ++p) {
            uint32_t *kout = (p % 2 == 0) ? s.keys_a : s.keys_b;
            uint32_t *vout = p == npass - 1 ? (uint32_t *)perm : ((p % 2 == 0) ? s.vals_a : s.vals_b);
            radix_pass(kin, vin, n, shift, widths[p], p > 0, items, s, kout, vout, mk, st);
            kin = kout;
            vin = vout;
            shift += widths[p];
        }
        *sorted_keys = kin;
    }
    const int sblk = (int)((n + 1 + kBlock - 1) / kBlock), cblk = (int)((g.ncell + 1 + kBlock - 1) / kBlock);
    mk->mark("segments", st);
    hipLaunchKernelGGL(k_segment_starts, dim3(sblk), dim3(kBlock), 0, st, *sorted_keys, n, g.ncell, start);
    hipLaunchKernelGGL(k_segment_counts, dim3(cblk), dim3(kBlock), 0, st, start, g.ncell, *sorted_keys, n, count);
    return hipGetLastError();
}

hipError_t launch_stable_partition(const uint32_t *keys, int64_t n, int bits, const SortScratch &s, uint32_t *keys_out,
                                   uint32_t *ids_out, hipStream_t st) {
    if (n <= 0) return hipGetLastError();
    Marker off;
    radix_pass(keys, nullptr, n, 0, bits, true, sort_items(n, s.max_tiles), s, keys_out, ids_out, &off, st);
    return hipGetLastError();
}

template hipError_t launch_bin_sort<float>(const float *, const float *, int64_t, const Geo<float> &, int32_t *,
                                           vec4<float> *, int32_t *, int32_t *, int32_t *, const SortScratch &,
                                           double *, const uint32_t **, Marker *, hipStream_t);
template hipError_t launch_bin_sort<double>(const double *, const double *, int64_t, const Geo<double> &, int32_t *,
                                            vec4<double> *, int32_t *, int32_t *, int32_t *, const SortScratch &,
                                            double *, const uint32_t **, Marker *, hipStream_t);

}  // namespace cpl
