// mlp.hip -- the learned velocity surrogate on the gfx950 matrix cores.
//
// The surrogate predicts the sub-bulk part of the fluid velocity at a particle
// (fine-grid lookup minus bulk trilinear interpolation) from the 3x3x3 bulk
// stencil around its cell, its in-cell offset and its diameter.  All products
// are v_mfma_f32_16x16x32_bf16: BF16 operands (rounded to nearest even), FP32
// accumulation.
//
// Operand layout of one 16x16x32 product on a 64-lane wave (lane l, n = l % 16,
// g = l / 16): the A operand lane holds row n and eight contraction slots of
// group g, the B operand lane holds column n and the same eight slots, and the
// result lane holds column n, rows 4g .. 4g+3.  Which contraction index a slot
// stands for is a labelling shared by A and B: any permutation works as long as
// both operands use it.
//
// Products are written "transposed": weights are the A operand (rows = output
// neurons), activations the B operand (columns = particles).  The result of one
// layer (column = particle, rows = neurons 4g..4g+3 of a 16-row block) is then
// already the B operand of the next layer once two row blocks are paired into
// one 32-wide slot group: slots 0-3 <- rows 32q+4g+j, slots 4-7 <- rows
// 32q+16+4g+j.  The in-step inference kernel chains the four layers this way in
// registers, with the weights pre-permuted into that slot order in LDS.
//
// The training pass chains forward and backward the same way, a 16-row tile
// per pair of waves, and writes transposed copies of the layer inputs and
// output gradients for the weight-gradient products, whose contraction runs
// over the batch.  Batch inference on given features chains the layers in
// registers too, in the natural slot order (rows k = 32q + 8g + i).  Every reduction has a fixed
// order.
#include <type_traits>

#include "common.hpp"
#include "launch.hpp"
#include "mlp.hpp"
#include "sample.hpp"

namespace cpl {
namespace mlp {

typedef __bf16 bf16x8 __attribute__((__vector_size__(16)));
typedef float f32x4 __attribute__((__vector_size__(16)));

// float -> bfloat16, round to nearest even (v_cvt_pk_bf16_f32 on gfx950).
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ uint32_t pack2(float lo, float hi) {
    const bf16x2 v = {(__bf16)lo, (__bf16)hi};
    return __builtin_bit_cast(uint32_t, v);
}
__device__ __forceinline__ uint32_t bf16_bits(float x) { return pack2(x, 0.f) & 0xffffu; }
__device__ __forceinline__ bf16x8 as_bf16x8(uint4 v) { return __builtin_bit_cast(bf16x8, v); }
__device__ __forceinline__ bf16x8 load8(const uint16_t *p) { return as_bf16x8(*reinterpret_cast<const uint4 *>(p)); }
__device__ __forceinline__ f32x4 mma(bf16x8 a, bf16x8 b, f32x4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}

// tanh-form GELU 0.5 z (1 + tanh(u)), u = sqrt(2/pi) (z + 0.044715 z^3), written
// as z * sigma(2u) with sigma(2u) = 1 / (1 + 2^(-2u log2 e)): one exp2 and one
// reciprocal (hardware, ~1 ulp).  For z -> -inf, 2^(...) -> inf and the result
// -> -0; for z -> +inf it -> z.  Derivative: with s = sigma(2u),
//   gelu'(z) = s + 2 z s (1 - s) du/dz,  du/dz = sqrt(2/pi) (1 + 3 * 0.044715 z^2).
constexpr float kGc = 0.7978845608028654f, kGa = 0.044715f;
constexpr float kGk = 2.3022081983914574f;   // 2 sqrt(2/pi) log2(e)
__device__ __forceinline__ float sig2u(float z) {
    const float t = fmaf(-kGk * kGa, z * z, -kGk);   // -2u log2(e) / z
    return __builtin_amdgcn_rcpf(1.f + __builtin_amdgcn_exp2f(z * t));
}
__device__ __forceinline__ float gelu(float z) { return z * sig2u(z); }

__device__ __forceinline__ int lane_id() { return threadIdx.x & (kWave - 1); }

// ---------------------------------------------------------------------------
// Parameter bookkeeping
// ---------------------------------------------------------------------------
// Flat parameter index -> (layer, is_weight, k, m).
__device__ __forceinline__ void decode_param(int64_t i, int &l, bool &w, int &k, int &m) {
    constexpr int64_t kW1 = off_w(1), kW2 = off_w(2), kW3 = off_w(3);
    constexpr int64_t kB0 = off_b(0), kB1 = off_b(1), kB2 = off_b(2), kB3 = off_b(3);
    l = i < kW1 ? 0 : (i < kW2 ? 1 : (i < kW3 ? 2 : 3));
    const int64_t w0 = l == 0 ? 0 : (l == 1 ? kW1 : (l == 2 ? kW2 : kW3));
    const int64_t b0 = l == 0 ? kB0 : (l == 1 ? kB1 : (l == 2 ? kB2 : kB3));
    const int fo = l == 3 ? kOut : kHid;
    w = i < b0;
    if (w) {
        k = (int)((i - w0) / fo);
        m = (int)((i - w0) % fo);
    } else {
        k = 0;
        m = (int)(i - b0);
    }
}

struct WPtrs {
    uint16_t *wt[4], *wn[4], *wtp[4], *wnp[4];
};

__device__ __forceinline__ void write_bf16_copies(const WPtrs &w, int l, int k, int m, float p) {
    const uint16_t b = (uint16_t)bf16_bits(p);
    w.wt[l][(int64_t)m * kpad(l) + k] = b;
    w.wtp[l][(int64_t)m * kpad(l) + (l == 0 ? slot_of_feature(k) : perm_col(k))] = b;
    if (l > 0) {
        w.wn[l][(int64_t)k * cpad(l) + m] = b;
        w.wnp[l][(int64_t)k * cpad(l) + perm_col(m)] = b;
    }
}

__global__ __launch_bounds__(kBlock) void k_cast(const float *__restrict__ params, WPtrs w) {
    const int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (i >= kNParam) return;
    int l, k, m;
    bool isw;
    decode_param(i, l, isw, k, m);
    if (isw) write_bf16_copies(w, l, k, m, params[i]);
}

// Adam (bias-corrected) on the FP32 master parameters, then the BF16 copies.
__global__ __launch_bounds__(kBlock) void k_adam(const float *__restrict__ grads, float *__restrict__ params,
                                                 float *__restrict__ mom1, float *__restrict__ mom2, WPtrs w,
                                                 float lr, float b1, float omb1, float b2, float omb2, float eps,
                                                 float c1, float c2) {
    const int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (i >= kNParam) return;
    const float g = grads[i];
    const float m = b1 * mom1[i] + omb1 * g;
    const float v = b2 * mom2[i] + omb2 * g * g;
    const float p = params[i] - lr * (m / c1) / (sqrtf(v / c2) + eps);
    mom1[i] = m;
    mom2[i] = v;
    params[i] = p;
    int l, k, mm;
    bool isw;
    decode_param(i, l, isw, k, mm);
    if (isw) write_bf16_copies(w, l, k, mm, p);
}

// ---------------------------------------------------------------------------
// Batch inference on given features
// ---------------------------------------------------------------------------
// The four layers in one pass over the features, which is all the memory traffic
// (layer by layer through memory, 50,001 rows took 108 us of kernels).  A
// workgroup of eight waves keeps the weights in LDS as product fragments (124
// KB) and loops over groups of 256 rows; a wave takes two 16-row tiles, whose
// activations stay in registers.  Slots are in the natural order (k = 32q + 8g +
// i), so a layer's result (lane group g: rows 4g .. 4g + 3 of a 16-row block)
// moves to the lane group that holds it in the next operand by two lane-swap
// instructions per word: see next_operand().
constexpr int kFwdWaves = 8, kFwdTiles = 2, kFwdRows = 16 * kFwdTiles * kFwdWaves;
constexpr int kFwdFrag1 = 8 * 7, kFwdFragH = 8 * 4, kFwdFrags = kFwdFrag1 + 2 * kFwdFragH + 4;

struct ForwardLds {
    uint4 frag[kFwdFrags][kWave];   // [neuron block][contraction block] of layers 1, 2, 3, then 4
    float bias[3 * kHid + 16];      // b1, b2, b3, b4 (padded)
    float mean[kK1], inv[kK1];
};

// Eight consecutive floats at any 4-byte address.
typedef float float4_u __attribute__((ext_vector_type(4), aligned(4)));

// Contraction block q of the next layer's operand from blocks 2q (a) and 2q + 1
// (b) of a result, two packed words each: lane group g takes rows 8g .. 8g + 7
// of the 32, rows 4g' .. 4g' + 3 of a 16-row block being in lane group g'.
// Swapping the upper 32 lanes of a with the lower 32 of b, then the odd 16-lane
// rows of the first with the even ones of the second, leaves the lower and the
// upper half of that run.
__device__ __forceinline__ uint4 next_operand(const uint32_t (&a)[2], const uint32_t (&b)[2]) {
    uint32_t lo[2], hi[2];
#pragma unroll
    for (int s = 0; s < 2; ++s) {
        const auto h = __builtin_amdgcn_permlane32_swap(a[s], b[s], false, false);
        const auto r = __builtin_amdgcn_permlane16_swap(h[0], h[1], false, false);
        lo[s] = r[0];
        hi[s] = r[1];
    }
    return make_uint4(lo[0], lo[1], hi[0], hi[1]);
}

// A hidden layer: in[t][kb] -> gelu(W in + b) -> out[t][4], natural slot order.
template <int KB>
__device__ __forceinline__ void forward_layer(const ForwardLds &L, int frag0, const float *bias,
                                              const uint4 (&in)[kFwdTiles][KB], uint4 (&out)[kFwdTiles][4], int lane,
                                              int g) {
    f32x4 acc[8][kFwdTiles];
#pragma unroll
    for (int mb = 0; mb < 8; ++mb)
#pragma unroll
        for (int t = 0; t < kFwdTiles; ++t) acc[mb][t] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int kb = 0; kb < KB; ++kb)
#pragma unroll
        for (int mb = 0; mb < 8; ++mb) {
            const bf16x8 w = as_bf16x8(L.frag[frag0 + mb * KB + kb][lane]);
#pragma unroll
            for (int t = 0; t < kFwdTiles; ++t) acc[mb][t] = mma(w, as_bf16x8(in[t][kb]), acc[mb][t]);
        }
#pragma unroll
    for (int q = 0; q < 4; ++q)
#pragma unroll
        for (int t = 0; t < kFwdTiles; ++t) {
            uint32_t h[2][2];
#pragma unroll
            for (int s = 0; s < 2; ++s) {
                const int mb = 2 * q + s;
                const float *bj = bias + 16 * mb + 4 * g;
                float z[4];
#pragma unroll
                for (int j = 0; j < 4; ++j) z[j] = acc[mb][t][j] + bj[j];
                h[s][0] = pack2(gelu(z[0]), gelu(z[1]));
                h[s][1] = pack2(gelu(z[2]), gelu(z[3]));
            }
            out[t][q] = next_operand(h[0], h[1]);
        }
}

struct ForwardNet {
    const uint16_t *wt[4];
    const float *params, *mean_inv;
};

// One layer's weights (rows of 32 KB BF16, 16 MB rows) into LDS as product
// fragments [neuron block][contraction block], 16 bytes per lane, by THREADS
// threads; all its loads are issued together.  (One loop over the fragments of
// all layers waits for the layer's address and then its weights, a fragment at a
// time: 26.5 us for the forward pass of 50,001 rows, 23.1 with all together.)
template <int KB, int MB, int THREADS>
__device__ __forceinline__ void stage_weights(const uint16_t *__restrict__ W, uint4 (*frag)[kWave]) {
    constexpr int kItems = MB * KB * kWave, kPer = (kItems + THREADS - 1) / THREADS;
    uint4 v[kPer];
#pragma unroll
    for (int i = 0; i < kPer; ++i) {
        const int e0 = threadIdx.x + i * THREADS, e = e0 < kItems ? e0 : 0;
        const int f = e >> 6, r = e & 15, gg = (e >> 4) & 3;
        v[i] = *reinterpret_cast<const uint4 *>(W + (16 * (f / KB) + r) * (32 * KB) + 32 * (f % KB) + 8 * gg);
    }
#pragma unroll
    for (int i = 0; i < kPer; ++i) {
        const int e = threadIdx.x + i * THREADS;
        if (e < kItems) frag[e >> 6][e & 63] = v[i];
    }
}

__global__ __launch_bounds__(kFwdWaves * kWave) void k_forward(const float *__restrict__ feat, int64_t B, ForwardNet net,
                                                               float *__restrict__ y) {
    __shared__ ForwardLds L;
    constexpr int NT = kFwdTiles, kThreads = kFwdWaves * kWave;
    const int lane = lane_id(), n = lane & 15, g = lane >> 4, wave = threadIdx.x >> 6;
    stage_weights<7, 8, kThreads>(net.wt[0], L.frag);
    stage_weights<4, 8, kThreads>(net.wt[1], L.frag + kFwdFrag1);
    stage_weights<4, 8, kThreads>(net.wt[2], L.frag + kFwdFrag1 + kFwdFragH);
    stage_weights<4, 1, kThreads>(net.wt[3], L.frag + kFwdFrag1 + 2 * kFwdFragH);
    for (int e = threadIdx.x; e < 3 * kHid + 16; e += kThreads) {
        const int l = e / kHid, m = e % kHid;
        constexpr int64_t kB0 = off_b(0), kB1 = off_b(1), kB2 = off_b(2), kB3 = off_b(3);
        L.bias[e] = l < 3 ? net.params[(l == 0 ? kB0 : (l == 1 ? kB1 : kB2)) + m] : (m < kOut ? net.params[kB3 + m] : 0.f);
    }
    for (int e = threadIdx.x; e < kK1; e += kThreads) {
        L.mean[e] = net.mean_inv[e];
        L.inv[e] = net.mean_inv[kK1 + e];
    }
    __syncthreads();
    for (int64_t b0 = (int64_t)blockIdx.x * kFwdRows + wave * 16 * NT; b0 < B; b0 += (int64_t)gridDim.x * kFwdRows) {
        // keeps the LDS reads below inside the loop (held in registers across
        // it, they would spill)
        wave_sync();
        // the rows' features (a row past the end: the last row, not stored), then
        // standardised into the layer-1 operand
        float v[NT][7][8];
#pragma unroll
        for (int t = 0; t < NT; ++t) {
            const int64_t b = b0 + 16 * t + n;
            const float *fr = feat + (b < B ? b : B - 1) * kFeat;
#pragma unroll
            for (int kb = 0; kb < 6; ++kb)
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    const float4_u q = *reinterpret_cast<const float4_u *>(fr + 32 * kb + 8 * g + 4 * h);
#pragma unroll
                    for (int i = 0; i < 4; ++i) v[t][kb][4 * h + i] = q[i];
                }
#pragma unroll
            for (int i = 0; i < 8; ++i) v[t][6][i] = 0.f;
            if (g == 0) v[t][6][0] = fr[192];   // the one feature of the last block
        }
        static_assert(kFeat == 193, "six whole contraction blocks and one feature");
        __builtin_amdgcn_sched_barrier(0);
        uint4 x[NT][7], h1[NT][4], h2[NT][4];
#pragma unroll
        for (int kb = 0; kb < 7; ++kb) {
#pragma unroll
            for (int t = 0; t < NT; ++t) {
                float s[8];
#pragma unroll
                for (int i = 0; i < 8; ++i) {
                    const int k = 32 * kb + 8 * g + i;
                    s[i] = kb < 6 || k < kFeat ? (v[t][kb][i] - L.mean[k]) * L.inv[k] : 0.f;
                }
                x[t][kb] = make_uint4(pack2(s[0], s[1]), pack2(s[2], s[3]), pack2(s[4], s[5]), pack2(s[6], s[7]));
            }
            __builtin_amdgcn_sched_barrier(0);   // a block at a time: the raw values go as the operand comes
        }
        __builtin_amdgcn_sched_barrier(0);
        forward_layer<7>(L, 0, L.bias, x, h1, lane, g);
        __builtin_amdgcn_sched_barrier(0);
        forward_layer<4>(L, kFwdFrag1, L.bias + kHid, h1, h2, lane, g);
        __builtin_amdgcn_sched_barrier(0);
        forward_layer<4>(L, kFwdFrag1 + kFwdFragH, L.bias + 2 * kHid, h2, h1, lane, g);
#pragma unroll
        for (int t = 0; t < NT; ++t) {
            f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int kb = 0; kb < 4; ++kb)
                acc = mma(as_bf16x8(L.frag[kFwdFrag1 + 2 * kFwdFragH + kb][lane]), as_bf16x8(h1[t][kb]), acc);
            const int64_t b = b0 + 16 * t + n;
            if (g == 0 && b < B)
#pragma unroll
                for (int j = 0; j < kOut; ++j) y[3 * b + j] = acc[j] + L.bias[3 * kHid + j];
        }
    }
}

// ---------------------------------------------------------------------------
// Training pass: standardisation, forward, loss and backward of 32 rows by a
// workgroup of four waves
// ---------------------------------------------------------------------------
// Batch rows are the product columns (lane n holds row 16 t + n of tile t) and
// neurons the product rows, as in the in-step inference.  A layer's result is
// the next B operand in the permuted slot order (slots 4s + j of group g <-
// neuron 32q + 16s + 4g + j); the weight fragments are read in the same order
// from the permuted copies, and the backward products take the output
// gradients in the same layout.  The four waves of a workgroup split every
// 128-neuron layer: wave w computes neuron blocks 2w and 2w + 1 (one
// contraction block q = w of the next product) for both 16-row tiles, so that
// each weight fragment it loads feeds two products, and keeps their gelu'(Z),
// formed in the forward pass with gelu (one exponential).  The other three
// contraction blocks of the next B operand are read back from the LDS stage
// below after a workgroup barrier; so is the layer-1 input, of which each wave
// loads and standardises two of the seven 32-feature blocks.  With an 80 KB
// stage and at most 256 registers per wave, two workgroups share a compute
// unit.
//
// For the weight-gradient products over the batch the pass writes the BF16
// layer inputs and the BF16 output gradients transposed, as the rows of one
// 1008-row matrix (x0 224, h 3 x 128, dZ 3 x 128 + 16) in blocks of 32 batch
// rows.  These are staged in LDS, [row][32 batch rows of the workgroup], and
// leave at the end as the workgroup's contiguous block: a wave's stores and
// loads share one in-order completion counter, so a store issued between the
// weight loads of two layers would make the second layer wait for it.  The
// bias gradients are the column sums of the FP32 output gradients: summed in
// FP64 over the 16 rows of a tile (a fixed butterfly), then over the two tiles
// of a workgroup in tile order, into part_b[l][workgroup][MP].  The loss
// partial of a tile is sum 0.5 (y - t)^2 / B.  B is a multiple of 32: every
// workgroup has both tiles.
constexpr int kTrainTiles = 2;                    // 16-row tiles per workgroup
static_assert(kTrainGroupRows == 16 * kTrainTiles, "two 16-row tiles per workgroup");
constexpr int kTrainWaves = 4;                    // a quarter of every layer's neurons each
constexpr int kTrainThreads = kTrainWaves * kWave;
constexpr int kBiasCols = 3 * kHid + 16;          // bias-gradient columns, layers 1-4
// Staged transposed rows: layer-1 input (224), hidden activations (3 x 128),
// output gradients (3 x 128 + 16).  36 BF16 per staged row: the four rows that
// one access instruction touches per lane group (4 apart) then fall 8 banks
// apart.
constexpr int kStagePitch = kTrainGroupRows + 4;
constexpr int kStageHt = kTrHt, kStageDz = kTrDz, kStageRows = kTrRows;
static_assert(kStageRows % 16 == 0, "the output pass takes whole rows");

struct TrainArgs {
    const float *feat, *resid;
    const int32_t *idx;
    int64_t nrows, B;
    const float *mean_inv;
    float is[3], inv_b;
    const float *params;
    const uint16_t *wt0;              // layer-1 W^T, natural order
    const uint16_t *wtp[4], *wnp[4];  // layers 2-4, permuted order
    uint16_t *tr;   // transposed rows, blocks of kTrBlock batch rows
    double *part_b[4];
    double *loss_part;
};

// Four BF16 values (two packed words) of column col staged to rows r0 .. r0+3.
__device__ __forceinline__ void stage_t4(uint16_t *S, int r0, int col, uint32_t w0, uint32_t w1) {
    S[r0 * kStagePitch + col] = (uint16_t)(w0 & 0xffffu);
    S[(r0 + 1) * kStagePitch + col] = (uint16_t)(w0 >> 16);
    S[(r0 + 2) * kStagePitch + col] = (uint16_t)(w1 & 0xffffu);
    S[(r0 + 3) * kStagePitch + col] = (uint16_t)(w1 >> 16);
}
// The same four values read back as two packed words.
__device__ __forceinline__ void unstage_t4(const uint16_t *S, int r0, int col, uint32_t &w0, uint32_t &w1) {
    w0 = (uint32_t)S[r0 * kStagePitch + col] | ((uint32_t)S[(r0 + 1) * kStagePitch + col] << 16);
    w1 = (uint32_t)S[(r0 + 2) * kStagePitch + col] | ((uint32_t)S[(r0 + 3) * kStagePitch + col] << 16);
}

// Sum over the 16 lanes of a lane group (lanes with equal g), FP64.
__device__ __forceinline__ double sum16(double v) {
#pragma unroll
    for (int o = 1; o < 16; o <<= 1) v += __shfl_xor(v, o, kWave);
    return v;
}

// Column sums over the 16 lanes of a lane group of the 8 values v = 4 b + j of
// a lane (FP32 in, FP64 sums): a reduce-scatter butterfly over lane bits 3, 2,
// 1 (each stage keeps half of the values, the upper half where the lane bit is
// set, adds the partner's copy of that half and sends the other half), then
// lanes n and n ^ 1 add their partial sums: both hold the sum of value n / 2.
// The adding order of every column is a fixed tree (a + b = b + a exactly, so
// partners agree).
__device__ __forceinline__ double colsum8(const float (&v)[8], int n) {
    double s4[4];
    const bool u3 = (n & 8) != 0;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const float recv = __shfl_xor(u3 ? v[i] : v[i + 4], 8, kWave);
        s4[i] = (double)(u3 ? v[i + 4] : v[i]) + (double)recv;
    }
    double s2[2];
    const bool u2 = (n & 4) != 0;
#pragma unroll
    for (int i = 0; i < 2; ++i) s2[i] = (u2 ? s4[i + 2] : s4[i]) + __shfl_xor(u2 ? s4[i] : s4[i + 2], 4, kWave);
    const bool u1 = (n & 2) != 0;
    const double s1 = (u1 ? s2[1] : s2[0]) + __shfl_xor(u1 ? s2[0] : s2[1], 2, kWave);
    return s1 + __shfl_xor(s1, 1, kWave);
}

// A quarter of a layer's output gradient (FP32, result layout; tiles t, blocks
// 2w + b): the BF16 values staged transposed (S, columns 16 t + n) and kept as
// packed words, the bias column sums of each tile into
// bs[t][16 (2w + b) + 4 g + j].
__device__ __forceinline__ void emit_grad(const f32x4 (&d)[2][2], int w, int n, int g, uint16_t *S,
                                          double (*bs)[kBiasCols], int bcol, uint32_t (&wv)[2][2][2]) {
#pragma unroll
    for (int t = 0; t < 2; ++t) {
        float v[8];
#pragma unroll
        for (int b = 0; b < 2; ++b) {
            wv[t][b][0] = pack2(d[t][b][0], d[t][b][1]);
            wv[t][b][1] = pack2(d[t][b][2], d[t][b][3]);
            stage_t4(S, 16 * (2 * w + b) + 4 * g, 16 * t + n, wv[t][b][0], wv[t][b][1]);
#pragma unroll
            for (int j = 0; j < 4; ++j) v[4 * b + j] = d[t][b][j];
        }
        const double cs = colsum8(v, n);   // value n / 2: block n / 8, row (n / 2) % 4
        if ((n & 1) == 0) bs[t][bcol + 16 * (2 * w + (n >> 3)) + 4 * g + ((n >> 1) & 3)] = cs;
    }
}

// A quarter of a hidden layer's result (tiles t, blocks 2w + b): Z = acc + b
// (bv: the bias values of the lane's rows), H = gelu(Z) as BF16 (staged
// transposed and kept as packed words), gelu'(Z) kept.
__device__ __forceinline__ void finish_hidden(const f32x4 (&acc)[2][2], const float4 (&bv)[2], int w, int n, int g,
                                              uint16_t *S, f32x4 (&gp)[2][2], uint32_t (&wv)[2][2][2]) {
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int b = 0; b < 2; ++b) {
            float hv[4];
            const float bj[4] = {bv[b].x, bv[b].y, bv[b].z, bv[b].w};
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const float z = acc[t][b][j] + bj[j];
                const float s = sig2u(z);
                hv[j] = z * s;   // gelu(z)
                gp[t][b][j] = s + 2.f * z * s * (1.f - s) * (kGc * fmaf(3.f * kGa, z * z, 1.f));   // gelu'(z)
            }
            wv[t][b][0] = pack2(hv[0], hv[1]);
            wv[t][b][1] = pack2(hv[2], hv[3]);
            stage_t4(S, 16 * (2 * w + b) + 4 * g, 16 * t + n, wv[t][b][0], wv[t][b][1]);
        }
}

// The full B operands (four contraction blocks, both tiles) of a 128-neuron
// result split over the four waves: block q = w from the wave's own packed
// words, the others read back from their staged rows (S).
__device__ __forceinline__ void gather_operand(const uint32_t (&wv)[2][2][2], const uint16_t *S, int w, int n, int g,
                                               bf16x8 (&x)[2][4]) {
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            uint32_t p[4];
            if (q == w) {
                p[0] = wv[t][0][0];
                p[1] = wv[t][0][1];
                p[2] = wv[t][1][0];
                p[3] = wv[t][1][1];
            } else {
                unstage_t4(S, 16 * (2 * q) + 4 * g, 16 * t + n, p[0], p[1]);
                unstage_t4(S, 16 * (2 * q + 1) + 4 * g, 16 * t + n, p[2], p[3]);
            }
            x[t][q] = as_bf16x8(make_uint4(p[0], p[1], p[2], p[3]));
        }
}

// A quarter of a 128 x 128 product in the permuted order: f[b][q] = row
// 16 (2w + b) + n of Mp (a permuted copy, pitch P), contraction block q, one
// 16-byte load.  A layer's fragments are loaded as one batch, ahead of the
// work before the product, so that their latency overlaps it; the product
// then runs on registers, each fragment feeding both tiles.
template <int P>
__device__ __forceinline__ void load_frags(const uint16_t *__restrict__ Mp, int w, int n, int g, bf16x8 (&f)[2][4]) {
#pragma unroll
    for (int b = 0; b < 2; ++b)
#pragma unroll
        for (int q = 0; q < 4; ++q) f[b][q] = load8(Mp + (16 * (2 * w + b) + n) * P + 32 * q + 8 * g);
}
// The bias values of a hidden layer for the lane's rows of blocks 2w, 2w + 1.
__device__ __forceinline__ void load_bias(const float *__restrict__ bias, int w, int g, float4 (&bv)[2]) {
#pragma unroll
    for (int b = 0; b < 2; ++b) bv[b] = *reinterpret_cast<const float4 *>(bias + 16 * (2 * w + b) + 4 * g);
}
__device__ __forceinline__ void product(const bf16x8 (&f)[2][4], const bf16x8 (&x)[2][4], f32x4 (&acc)[2][2]) {
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int b = 0; b < 2; ++b) {
            acc[t][b] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int q = 0; q < 4; ++q) acc[t][b] = mma(f[b][q], x[t][q], acc[t][b]);
        }
}
// Keeps the loads above it from sinking towards their first use.
__device__ __forceinline__ void issue_fence() { __builtin_amdgcn_sched_barrier(0); }

__global__ __launch_bounds__(kTrainThreads) __attribute__((amdgpu_waves_per_eu(2))) void k_train_tile(TrainArgs a) {
    __shared__ __align__(16) uint16_t stage[kStageRows * kStagePitch];
    __shared__ float norm[2 * kK1];
    __shared__ double bsum[kTrainTiles][kBiasCols];
    constexpr int64_t kOffB0 = off_b(0), kOffB1 = off_b(1), kOffB2 = off_b(2), kOffB3 = off_b(3);
    const int lane = lane_id(), n = lane & 15, g = lane >> 4;
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int64_t tile0 = (int64_t)blockIdx.x * kTrainTiles;
    uint16_t *sh = stage + kStageHt * kStagePitch, *sd = stage + kStageDz * kStagePitch;
    f32x4 acc[2][2], gp[3][2][2];
    uint32_t wv[2][2][2];
    bf16x8 x[2][4], f[2][4];
    float4 bv[2];

    // The standardisation table, the row numbers of both tiles and the layer-1
    // weight fragments of this wave's neuron blocks; then, from the row numbers,
    // the rows' residuals and the wave's share of their features, blocks kb = 2w,
    // 2w + 1 (< 7): two memory round trips.  No load is conditional: one that is
    // waits for those before it, and the rows element by element, tile after
    // tile, made nine round trips of the two (114 us for 65,536 rows).
    float t[2][4];
    {
        constexpr int kNormPer = (2 * kK1 + kTrainThreads - 1) / kTrainThreads;
        float nv[kNormPer];
#pragma unroll
        for (int i = 0; i < kNormPer; ++i) {
            const int e = threadIdx.x + i * kTrainThreads;
            nv[i] = a.mean_inv[e < 2 * kK1 ? e : 0];
        }
        int64_t row[2];
#pragma unroll
        for (int tt = 0; tt < 2; ++tt) row[tt] = (tile0 + tt) * 16 + n;
        if (a.idx) {   // uniform over the launch
            const int32_t r0 = a.idx[row[0]], r1 = a.idx[row[1]];
            row[0] = r0;
            row[1] = r1;
        }
        bf16x8 f1[2][7];
#pragma unroll
        for (int b = 0; b < 2; ++b)
#pragma unroll
            for (int kb = 0; kb < 7; ++kb) f1[b][kb] = load8(a.wt0 + (16 * (2 * w + b) + n) * kK1 + 32 * kb + 8 * g);
        issue_fence();
        float fv[2][2][8], rv[2][kOut];
#pragma unroll
        for (int tt = 0; tt < 2; ++tt) {
            if (row[tt] < 0 || row[tt] >= a.nrows) row[tt] = 0;   // documented: indices must be in range; keeps loads in bounds
#pragma unroll
            for (int j = 0; j < kOut; ++j) rv[tt][j] = a.resid[row[tt] * 3 + j];
        }
        if (w < 3) {   // uniform over the wave: blocks 2w, 2w + 1 <= 5 are whole
#pragma unroll
            for (int tt = 0; tt < 2; ++tt)
#pragma unroll
                for (int kk = 0; kk < 2; ++kk)
#pragma unroll
                    for (int h = 0; h < 2; ++h) {
                        const float4_u q = *reinterpret_cast<const float4_u *>(a.feat + row[tt] * kFeat +
                                                                              32 * (2 * w + kk) + 8 * g + 4 * h);
#pragma unroll
                        for (int i = 0; i < 4; ++i) fv[tt][kk][4 * h + i] = q[i];
                    }
        } else {       // block 6: feature 192 alone
#pragma unroll
            for (int tt = 0; tt < 2; ++tt) {
                const float q = a.feat[row[tt] * kFeat + kFeat - 1];
#pragma unroll
                for (int kk = 0; kk < 2; ++kk)
#pragma unroll
                    for (int i = 0; i < 8; ++i) fv[tt][kk][i] = (kk == 0 && i == 0 && g == 0) ? q : 0.f;
            }
        }
        issue_fence();
#pragma unroll
        for (int i = 0; i < kNormPer; ++i) {
            const int e = threadIdx.x + i * kTrainThreads;
            if (e < 2 * kK1) norm[e] = nv[i];
        }
        __syncthreads();   // the standardisation table
#pragma unroll
        for (int tt = 0; tt < 2; ++tt)
#pragma unroll
            for (int j = 0; j < 4; ++j) t[tt][j] = (g == 0 && j < kOut) ? rv[tt][j < kOut ? j : 0] * a.is[j < kOut ? j : 0] : 0.f;
        issue_fence();
#pragma unroll
        for (int tt = 0; tt < 2; ++tt)
#pragma unroll
            for (int kk = 0; kk < 2; ++kk) {
                const int kb = 2 * w + kk;
                if (kb < 7) {
                    float v[8];
#pragma unroll
                    for (int i = 0; i < 8; ++i) {
                        const int k = 32 * kb + 8 * g + i;
                        v[i] = k < kFeat ? (fv[tt][kk][i] - norm[k]) * norm[kK1 + k] : 0.f;
                    }
                    stage_t4(stage, 32 * kb + 8 * g, 16 * tt + n, pack2(v[0], v[1]), pack2(v[2], v[3]));
                    stage_t4(stage, 32 * kb + 8 * g + 4, 16 * tt + n, pack2(v[4], v[5]), pack2(v[6], v[7]));
                }
            }
        __syncthreads();   // the layer-1 input staged
#pragma unroll
        for (int tt = 0; tt < 2; ++tt) {
            bf16x8 xb[7];
#pragma unroll
            for (int kb = 0; kb < 7; ++kb) {
                uint32_t p[4];
                unstage_t4(stage, 32 * kb + 8 * g, 16 * tt + n, p[0], p[1]);
                unstage_t4(stage, 32 * kb + 8 * g + 4, 16 * tt + n, p[2], p[3]);
                xb[kb] = as_bf16x8(make_uint4(p[0], p[1], p[2], p[3]));
            }
#pragma unroll
            for (int b = 0; b < 2; ++b) {
                acc[tt][b] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int kb = 0; kb < 7; ++kb) acc[tt][b] = mma(f1[b][kb], xb[kb], acc[tt][b]);
            }
        }
    }
    load_frags<kHid>(a.wtp[1], w, n, g, f);
    load_bias(a.params + kOffB0, w, g, bv);
    issue_fence();
    finish_hidden(acc, bv, w, n, g, sh, gp[0], wv);
    __syncthreads();   // layer 1 staged
    gather_operand(wv, sh, w, n, g, x);
    product(f, x, acc);
    load_frags<kHid>(a.wtp[2], w, n, g, f);
    load_bias(a.params + kOffB1, w, g, bv);
    issue_fence();
    finish_hidden(acc, bv, w, n, g, sh + kHid * kStagePitch, gp[1], wv);
    __syncthreads();   // layer 2 staged
    gather_operand(wv, sh + kHid * kStagePitch, w, n, g, x);
    product(f, x, acc);
    bf16x8 fo[4], f4[2];
#pragma unroll
    for (int q = 0; q < 4; ++q) fo[q] = load8(a.wtp[3] + n * kHid + 32 * q + 8 * g);
#pragma unroll
    for (int b = 0; b < 2; ++b) f4[b] = load8(a.wnp[3] + (16 * (2 * w + b) + n) * 32 + 8 * g);
    load_bias(a.params + kOffB2, w, g, bv);
    float yb[4] = {0.f, 0.f, 0.f, 0.f};   // output bias of the lane's rows m = 4 g + j
#pragma unroll
    for (int j = 0; j < kOut; ++j) {
        const float q = a.params[kOffB3 + j];
        yb[j] = g == 0 ? q : 0.f;
    }
    issue_fence();
    finish_hidden(acc, bv, w, n, g, sh + 2 * kHid * kStagePitch, gp[2], wv);
    __syncthreads();   // layer 3 staged
    gather_operand(wv, sh + 2 * kHid * kStagePitch, w, n, g, x);

    // output layer (rows m = 4 g + j, three of them real) in every wave; the
    // loss, dY's staged rows and its bias sums from wave 0
    double lp[2];
    bf16x8 dy[2];
#pragma unroll
    for (int tt = 0; tt < 2; ++tt) {
        f32x4 y = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int q = 0; q < 4; ++q) y = mma(fo[q], x[tt][q], y);
        float d[4];
        lp[tt] = 0.0;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int m = 4 * g + j;
            const float dd = m < kOut ? (y[j] + yb[j]) - t[tt][j] : 0.f;
            lp[tt] += 0.5 * (double)dd * (double)dd;
            d[j] = dd * a.inv_b;
        }
        const uint32_t w0 = pack2(d[0], d[1]), w1 = pack2(d[2], d[3]);
        dy[tt] = as_bf16x8(make_uint4(w0, w1, 0u, 0u));
        if (w == 0) {
            stage_t4(sd + 3 * kHid * kStagePitch, 4 * g, 16 * tt + n, w0, w1);
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const double s = sum16((double)d[j]);
                if (n == 0) bsum[tt][3 * kHid + 4 * g + j] = s;
            }
        }
    }
    // backward: dZ_l = (dZ_{l+1} W_{l+1}^T) .* gelu'(Z_l), l = 3, 2, 1
#pragma unroll
    for (int tt = 0; tt < 2; ++tt)
#pragma unroll
        for (int b = 0; b < 2; ++b) {
            acc[tt][b] = mma(f4[b], dy[tt], f32x4{0.f, 0.f, 0.f, 0.f});
            acc[tt][b] *= gp[2][tt][b];
        }
    load_frags<kHid>(a.wnp[2], w, n, g, f);
    issue_fence();
    emit_grad(acc, w, n, g, sd + 2 * kHid * kStagePitch, bsum, 2 * kHid, wv);
    __syncthreads();   // dZ3 staged
    gather_operand(wv, sd + 2 * kHid * kStagePitch, w, n, g, x);
    product(f, x, acc);
#pragma unroll
    for (int tt = 0; tt < 2; ++tt)
#pragma unroll
        for (int b = 0; b < 2; ++b) acc[tt][b] *= gp[1][tt][b];
    load_frags<kHid>(a.wnp[1], w, n, g, f);
    issue_fence();
    emit_grad(acc, w, n, g, sd + kHid * kStagePitch, bsum, kHid, wv);
    __syncthreads();   // dZ2 staged
    gather_operand(wv, sd + kHid * kStagePitch, w, n, g, x);
    product(f, x, acc);
#pragma unroll
    for (int tt = 0; tt < 2; ++tt)
#pragma unroll
        for (int b = 0; b < 2; ++b) acc[tt][b] *= gp[0][tt][b];
    emit_grad(acc, w, n, g, sd, bsum, 0, wv);
#pragma unroll
    for (int tt = 0; tt < 2; ++tt) {
        const double l = wave_sum(lp[tt]);
        if (lane == 0 && w == 0) a.loss_part[tile0 + tt] = l * (double)a.inv_b;
    }
    __syncthreads();   // the group is staged
    for (int c = threadIdx.x; c < kBiasCols; c += kTrainThreads) {
        const double sb = bsum[0][c] + bsum[1][c];
        const int l = c < 3 * kHid ? c / kHid : 3, m = c - l * kHid, MP = mpad(l);
        a.part_b[l][(int64_t)blockIdx.x * MP + m] = sb;
    }
    // the staged block out: kTrRows rows of 32 batch rows, 8 threads per row
    // with 4 batch rows (8 bytes) each
    uint16_t *dst = a.tr + (int64_t)blockIdx.x * kStageRows * kTrBlock;
    constexpr int kChunks = kStageRows * kTrBlock / 4, kU = 8;
    constexpr int kIter = (kChunks + kTrainThreads - 1) / kTrainThreads;
    for (int i0 = 0; i0 < kIter; i0 += kU) {
        uint2 v[kU];
#pragma unroll
        for (int u = 0; u < kU; ++u) {
            const int e = threadIdx.x + kTrainThreads * (i0 + u);
            if (e < kChunks) v[u] = *reinterpret_cast<const uint2 *>(stage + (e >> 3) * kStagePitch + 4 * (e & 7));
        }
#pragma unroll
        for (int u = 0; u < kU; ++u) {
            const int e = threadIdx.x + kTrainThreads * (i0 + u);
            if (e < kChunks) *reinterpret_cast<uint2 *>(dst + 4 * e) = v[u];
        }
    }
}

// Weight gradients of one layer over a chunk of rows:
//   part_w[c][m][k] = sum_{b in chunk} dZ[b][m] H[b][k]   (BF16 x BF16, FP32 accumulate)
// from the training pass's transposed rows (dZ rows dz_row + 16 MT, H rows
// h_row + 16 KT, blocks of kTrBlock batch rows).  Rows in chunks of kChunk; B
// is a multiple of 32.  A wave takes NK output column blocks from kt on and
// keeps all MT row blocks of each in registers: per 32 rows it loads NK H
// fragments and the MT dZ fragments and issues NK MT independent products.  The
// fragment loads bound it (a dZ fragment is read once per wave of its layer):
// with one column block per wave they were 9 for 8 products (49 us for 65,536
// rows), with two they are 10 for 16 (35.9 us); unrolled over the 256 rows of a chunk
// instead of 128, 33.5 us.  The compiler moves the loads down to their products: its 94
// registers (five waves per SIMD) are the 64 sums and some seven fragments.
template <int MT, int KT, int NK>
__device__ __forceinline__ void wgrad_chunk(const uint16_t *__restrict__ tr, int dz_row, int h_row, int64_t B, int kt,
                                            float *__restrict__ part_w) {
    constexpr int MP = 16 * MT, KP = 16 * KT;
    constexpr int64_t kBlk = (int64_t)kTrRows * kTrBlock;   // elements per block of batch rows
    static_assert(kTrBlock == 32, "one block per 32-row product");
    const int lane = lane_id(), n = lane & 15, g = lane >> 4;
    const int64_t c = blockIdx.x;
    const int64_t b0 = c * kChunk, b1 = (b0 + kChunk < B) ? b0 + kChunk : B;
    f32x4 acc[NK][MT];
#pragma unroll
    for (int k = 0; k < NK; ++k)
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) acc[k][mt] = f32x4{0.f, 0.f, 0.f, 0.f};
    const uint16_t *pb = tr + (int64_t)(h_row + 16 * kt + n) * kTrBlock + 8 * g;
    const uint16_t *pa = tr + (int64_t)(dz_row + n) * kTrBlock + 8 * g;
    // kU groups of 32 rows per round (the rows are summed in order)
    constexpr int kU = 8;
    for (int64_t bb = b0; bb < b1; bb += 32 * kU) {
        bf16x8 bv[kU][NK];
        bf16x8 av[kU][MT];
#pragma unroll
        for (int u = 0; u < kU; ++u) {
            const int64_t r = bb + 32 * u < b1 ? bb + 32 * u : b1 - 32;
            const int64_t o = (r / kTrBlock) * kBlk;
#pragma unroll
            for (int k = 0; k < NK; ++k) bv[u][k] = load8(pb + 16 * k * kTrBlock + o);
#pragma unroll
            for (int mt = 0; mt < MT; ++mt) av[u][mt] = load8(pa + 16 * mt * kTrBlock + o);
        }
#pragma unroll
        for (int u = 0; u < kU; ++u) {
            if (bb + 32 * u >= b1) break;
#pragma unroll
            for (int mt = 0; mt < MT; ++mt)
#pragma unroll
                for (int k = 0; k < NK; ++k) acc[k][mt] = mma(av[u][mt], bv[u][k], acc[k][mt]);
        }
    }
#pragma unroll
    for (int k = 0; k < NK; ++k)
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) {
            float *o = part_w + (c * MP + 16 * mt + 4 * g) * KP + 16 * (kt + k) + n;
#pragma unroll
            for (int j = 0; j < 4; ++j) o[(int64_t)j * KP] = acc[k][mt][j];
        }
}

// The four layers' weight gradients in one launch.  Of the eight waves of
// workgroup (chunk, 0) seven take layer 1's fourteen column blocks and one the
// eight of layer 4 (one row block each); those of (chunk, 1) take the eight of
// layer 2 and of layer 3.
constexpr int kWgradWaves = 8;
struct WgradParts {
    float *w[4];
};
__global__ __launch_bounds__(kWgradWaves * kWave) void k_wgrad(const uint16_t *__restrict__ tr, int64_t B,
                                                               WgradParts parts) {
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    if (blockIdx.y == 0) {
        if (w < 7) wgrad_chunk<8, 14, 2>(tr, kTrDz, 0, B, 2 * w, parts.w[0]);
        else wgrad_chunk<1, 8, 8>(tr, kTrDz + 3 * kHid, kTrHt + 2 * kHid, B, 0, parts.w[3]);
    } else if (w < 4) {
        wgrad_chunk<8, 8, 2>(tr, kTrDz + kHid, kTrHt, B, 2 * w, parts.w[1]);
    } else {
        wgrad_chunk<8, 8, 2>(tr, kTrDz + 2 * kHid, kTrHt + kHid, B, 2 * (w - 4), parts.w[2]);
    }
}

struct GradParts {
    const float *w[4];
    const double *b[4];
};

// Flat gradient vector and loss from the partials, in one launch: a workgroup for
// the loss, kRedBBlocks for the bias entries (the longest chains first) and
// kRedWBlocks for the weight entries (three launches of which two do not fill the
// chip took 24 us of a 65,536-row step).
//
// Weight entries follow the partials' layout (per layer the padded [m][k] slots,
// k fastest), so that the loads of a wave are contiguous; each is summed by
// kRedGroups threads over interleaved chunks (c mod kRedGroups, two partial sums
// each) whose results are combined in a fixed order.
constexpr int kRedThreads = 1024;
constexpr int kRedGroups = 8;
constexpr int kRedEntries = kRedThreads / kRedGroups;   // weight entries per workgroup
constexpr int64_t kRedW1 = (int64_t)mpad(0) * kpad(0), kRedW2 = kRedW1 + (int64_t)mpad(1) * kpad(1),
                  kRedW3 = kRedW2 + (int64_t)mpad(2) * kpad(2), kRedTotal = kRedW3 + (int64_t)mpad(3) * kpad(3);
// Bias entries are summed over the workgroup partials of the training pass:
// kRedBEntries consecutive entries per workgroup, kRedBLanes threads per entry
// over interleaved partials (c mod kRedBLanes; a wave reads 8 partials of 8
// consecutive entries), then one thread per entry adds the lanes' sums in order.
constexpr int kRedBias = 3 * kHid + kOut;          // bias entries (real ones)
constexpr int kRedBEntries = 8, kRedBLanes = kRedThreads / kRedBEntries;
constexpr int kRedWBlocks = (int)((kRedTotal + kRedEntries - 1) / kRedEntries);
constexpr int kRedBBlocks = (kRedBias + kRedBEntries - 1) / kRedBEntries;

// Sum of p[c stride] over c = first, first + step, ... < count in two alternating
// partial sums (even and odd terms), eight loads at a time.
template <typename P>
__device__ __forceinline__ double strided_sum(const P *__restrict__ p, int64_t stride, int64_t first, int64_t step,
                                              int64_t count) {
    constexpr int kU = 8;
    double s[2] = {0.0, 0.0};
    int64_t c = first;
    for (; c + (kU - 1) * step < count; c += kU * step) {
        P v[kU];
#pragma unroll
        for (int u = 0; u < kU; ++u) v[u] = p[(c + u * step) * stride];
#pragma unroll
        for (int u = 0; u < kU; ++u) s[u & 1] += (double)v[u];
    }
    for (int u = 0; c < count; c += step, u ^= 1) s[u] += (double)p[c * stride];
    return s[0] + s[1];
}

__device__ __forceinline__ void reduce_weights(const GradParts &parts, int64_t nchunk, int block, double *red,
                                               float *__restrict__ grads) {
    constexpr int64_t kOffW[4] = {off_w(0), off_w(1), off_w(2), off_w(3)};
    const int le = threadIdx.x % kRedEntries, grp = threadIdx.x / kRedEntries;
    const int64_t e = (int64_t)block * kRedEntries + le;
    const int l = e < kRedW1 ? 0 : (e < kRedW2 ? 1 : (e < kRedW3 ? 2 : 3));
    const int64_t r = e - (l == 0 ? 0 : (l == 1 ? kRedW1 : (l == 2 ? kRedW2 : kRedW3)));
    const int MP = l == 3 ? mpad(3) : kHid, KP = l == 0 ? kpad(0) : kHid;
    const int m = (int)(r / KP), k = (int)(r % KP);
    red[grp * kRedEntries + le] =
        e < kRedTotal ? strided_sum(parts.w[l] + r, (int64_t)MP * KP, grp, kRedGroups, nchunk) : 0.0;
    __syncthreads();
    if (grp == 0 && e < kRedTotal) {
        double t = 0.0;
#pragma unroll
        for (int q = 0; q < kRedGroups; ++q) t += red[q * kRedEntries + le];
        const int fi = l == 0 ? kFeat : kHid, fo = l == 3 ? kOut : kHid;
        if (k < fi && m < fo) grads[kOffW[l] + (int64_t)k * fo + m] = (float)t;
    }
}

__device__ __forceinline__ void reduce_biases(const GradParts &parts, int64_t nchunk_b, int block, double *red,
                                              float *__restrict__ grads) {
    constexpr int64_t kOffB[4] = {off_b(0), off_b(1), off_b(2), off_b(3)};
    const int le = threadIdx.x % kRedBEntries, cl = threadIdx.x / kRedBEntries;
    const int e = block * kRedBEntries + le;
    const int l = e < 3 * kHid ? e / kHid : 3, m = e - l * kHid, MP = mpad(l);
    red[cl * kRedBEntries + le] = e < kRedBias ? strided_sum(parts.b[l] + m, MP, cl, kRedBLanes, nchunk_b) : 0.0;
    __syncthreads();
    if (cl == 0 && e < kRedBias) {
        double t = 0.0;
        for (int q = 0; q < kRedBLanes; ++q) t += red[q * kRedBEntries + le];
        grads[kOffB[l] + m] = (float)t;
    }
}

__device__ __forceinline__ void reduce_loss(const double *__restrict__ part, int64_t n, double *red,
                                            float *__restrict__ out) {
    double v = 0.0;
    if (threadIdx.x < kBlock) {   // whole waves
        constexpr int kU = 16;   // loads at a time
        int64_t i = threadIdx.x;
        for (; i + (kU - 1) * kBlock < n; i += kU * kBlock) {
            double p[kU];
#pragma unroll
            for (int u = 0; u < kU; ++u) p[u] = part[i + u * kBlock];
#pragma unroll
            for (int u = 0; u < kU; ++u) v += p[u];
        }
        for (; i < n; i += kBlock) v += part[i];
        v = wave_sum(v);
        if (threadIdx.x % kWave == 0) red[threadIdx.x / kWave] = v;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        double t = 0.0;
        for (int q = 0; q < kWavesPerBlock; ++q) t += red[q];
        out[0] = (float)t;
    }
}

__global__ __launch_bounds__(kRedThreads) void k_reduce(GradParts parts, int64_t nchunk, int64_t nchunk_b,
                                                        float *__restrict__ grads,
                                                        const double *__restrict__ loss_part, int64_t nloss,
                                                        float *__restrict__ loss) {
    __shared__ double red[kRedThreads];
    const int b = blockIdx.x - (loss ? 1 : 0);
    if (b < 0) reduce_loss(loss_part, nloss, red, loss);
    else if (b < kRedBBlocks) reduce_biases(parts, nchunk_b, b, red, grads);
    else reduce_weights(parts, nchunk, b - kRedBBlocks, red, grads);
}

// Column statistics: pass 0 sums x, pass 1 sums (x - mean)^2, per chunk of rows.
__global__ __launch_bounds__(kBlock) void k_colsum(const float *__restrict__ x, int64_t n, int cols, int64_t rows_per,
                                                   const double *__restrict__ mean, double *__restrict__ part) {
    const int c = threadIdx.x;
    if (c >= cols) return;
    const int64_t r0 = (int64_t)blockIdx.x * rows_per, r1 = (r0 + rows_per < n) ? r0 + rows_per : n;
    const double mu = mean ? mean[c] : 0.0;
    double s = 0.0;
    for (int64_t r = r0; r < r1; ++r) {
        const double v = (double)x[r * cols + c] - mu;
        s += mean ? v * v : v;
    }
    part[(int64_t)blockIdx.x * cols + c] = s;
}

__global__ __launch_bounds__(kBlock) void k_colfinish(const double *__restrict__ part, int64_t nchunk, int cols,
                                                      int64_t n, int sq, double *__restrict__ out) {
    const int c = threadIdx.x;
    if (c >= cols) return;
    double s = 0.0;
    for (int64_t k = 0; k < nchunk; ++k) s += part[k * cols + c];
    out[c] = sq ? sqrt(s / (double)n) : s / (double)n;
}

// ---------------------------------------------------------------------------
// Features of given particles from the bulk fields (training pairs)
// ---------------------------------------------------------------------------
// feat[j] = the 193 raw features of particle i = sel[j] (or j): per stencil cell
// (dz, dy, dx in -1..1, dx fastest, clamped at the walls) eps = 1 - phi, U, G,
// neighbours minus the centre cell; offsets x * n / L - i; d * n_x / L_x.
// u_bulk[j] = bulk trilinear velocity; resid[j] = u_fine[i] - u_bulk[j].
__global__ __launch_bounds__(kBlock) void k_features(Geo<float> g, int64_t n, const float *__restrict__ pos,
                                                     const float *__restrict__ diam, const float *__restrict__ phi,
                                                     const float *__restrict__ U, const float *__restrict__ G,
                                                     const float *__restrict__ u_fine, const int32_t *__restrict__ sel,
                                                     int64_t nsel, float *__restrict__ feat,
                                                     float *__restrict__ u_bulk, float *__restrict__ resid) {
    const int64_t j = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (j >= nsel) return;
    int64_t i = sel ? (int64_t)sel[j] : j;
    if (i < 0 || i >= n) i = 0;   // documented: entries must be in range; keeps loads in bounds
    int o = 0;
    const float x = clamp_coord(pos[3 * i + 0], g.L[0], o), y = clamp_coord(pos[3 * i + 1], g.L[1], o),
                z = clamp_coord(pos[3 * i + 2], g.L[2], o);
    const int ix = cell_axis(x, g.sb[0], g.nb[0]), iy = cell_axis(y, g.sb[1], g.nb[1]),
              iz = cell_axis(z, g.sb[2], g.nb[2]);
    const int64_t nx = g.nb[0], nxy = (int64_t)g.nb[0] * g.nb[1], nc = g.ncell;
    const int64_t c0 = ix + nx * iy + nxy * iz;
    float cen[7] = {1.f - phi[c0], U[c0], U[nc + c0], U[2 * nc + c0], G[c0], G[nc + c0], G[2 * nc + c0]};
    float *out = feat + j * kFeat;
    int col = 0;
    for (int dz = -1; dz <= 1; ++dz)
        for (int dy = -1; dy <= 1; ++dy)
            for (int dx = -1; dx <= 1; ++dx) {
                const int cx = clampi(ix + dx, g.nb[0]), cy = clampi(iy + dy, g.nb[1]), cz = clampi(iz + dz, g.nb[2]);
                const int64_t c = cx + nx * cy + nxy * cz;
                const float v[7] = {1.f - phi[c], U[c], U[nc + c], U[2 * nc + c], G[c], G[nc + c], G[2 * nc + c]};
                const bool centre = (dx == 0 && dy == 0 && dz == 0);
                for (int k = 0; k < 7; ++k) out[col++] = centre ? cen[k] : v[k] - cen[k];
            }
    out[col++] = x * g.sb[0] - (float)ix;
    out[col++] = y * g.sb[1] - (float)iy;
    out[col++] = z * g.sb[2] - (float)iz;
    out[col++] = diam[i] * g.sb[0];
    if (u_bulk || resid) {
        const Axis<float> bx = cic_axis(x, g.sb[0], g.nb[0]);
        const Axis<float> by = cic_axis(y, g.sb[1], g.nb[1]);
        const Axis<float> bz = cic_axis(z, g.sb[2], g.nb[2]);
        const int inx = g.nb[0];
        float ub[3];
        for (int a = 0; a < 3; ++a) ub[a] = trilin_pairs(U + a * nc, bx, by, bz, inx, nxy);
        if (u_bulk)
            for (int a = 0; a < 3; ++a) u_bulk[3 * j + a] = ub[a];
        if (resid && u_fine)
            for (int a = 0; a < 3; ++a) resid[3 * j + a] = u_fine[3 * i + a] - ub[a];
    }
}

// ---------------------------------------------------------------------------
// In-step inference: packed bulk features, fused gather + four-layer chain,
// sampled check with fine fallback
// ---------------------------------------------------------------------------
// fgrid[2c] = (1 - phi, U_x, U_y, U_z), fgrid[2c+1] = (G_x, G_y, G_z, 0); G is
// also written to the bulk gradient output (same values as the source stage).
__global__ __launch_bounds__(kBlock) void k_pack(StepArgs<float> a) {
    const int64_t c = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (c >= a.g.ncell) return;
    int cx, cy, cz;
    decode_cell(c, a.g.nb, cx, cy, cz);
    float gr[3];
    gradient_at(c, cx, cy, cz, a.g.nb, a.g.hb, a.P, a.Plo, gr);
    const int64_t nc = a.g.ncell;
    for (int k = 0; k < 3; ++k) a.G[k * nc + c] = gr[k];
    a.fgrid[2 * c] = make_float4(1.f - a.phi[c], a.U[c], a.U[nc + c], a.U[2 * nc + c]);
    a.fgrid[2 * c + 1] = make_float4(gr[0], gr[1], gr[2], 0.f);
}

constexpr int kInfWaves = 8;                    // waves per workgroup (two per SIMD: the LDS and 256 VGPRs per wave)
constexpr int kInfTiles = 2;                    // 16-particle tiles per wave and round
constexpr int kInfRows = 16 * kInfTiles;        // particles per wave and round
constexpr int kFrag1 = 8 * 7, kFragH = 8 * 4;   // operand fragments per layer
constexpr int kFrags = kFrag1 + 2 * kFragH + 4;

struct InferLds {
    uint4 frag[kFrags][kWave];    // weight fragments in slot order, 16 B per lane
    float bias[3 * kHid + 16];    // b1, b2, b3, b4 (padded)
    float mean[kK1], inv[kK1];    // standardisation per layer-1 slot (0 in the padding)
};

// One layer of the chain for NT tiles: in[t][kb] (KB slot groups) -> 8 row
// blocks (accumulators start at the bias) -> gelu -> out[t][4] in the paired
// slot order.  The slot-group loop is outermost so that the 8 NT accumulators
// form independent MFMA chains (a dependent MFMA waits for its predecessor);
// each weight fragment read from LDS feeds NT products.
template <int NT, int KB>
__device__ __forceinline__ void chain_layer(const InferLds &L, int frag0, const float *bias,
                                            const uint4 (&in)[NT][KB], uint4 (&out)[NT][4], int lane, int g) {
    f32x4 acc[8][NT];
#pragma unroll
    for (int mb = 0; mb < 8; ++mb) {
        const int m0 = 16 * mb + 4 * g;
        const f32x4 b = {bias[m0], bias[m0 + 1], bias[m0 + 2], bias[m0 + 3]};
#pragma unroll
        for (int t = 0; t < NT; ++t) acc[mb][t] = b;
    }
#pragma unroll
    for (int kb = 0; kb < KB; ++kb)
#pragma unroll
        for (int mb = 0; mb < 8; ++mb) {
            const bf16x8 w = as_bf16x8(L.frag[frag0 + mb * KB + kb][lane]);
#pragma unroll
            for (int t = 0; t < NT; ++t) acc[mb][t] = mma(w, as_bf16x8(in[t][kb]), acc[mb][t]);
        }
#pragma unroll
    for (int mb = 0; mb < 8; ++mb)
#pragma unroll
        for (int t = 0; t < NT; ++t) {
            const uint32_t lo = pack2(gelu(acc[mb][t][0]), gelu(acc[mb][t][1]));
            const uint32_t hi = pack2(gelu(acc[mb][t][2]), gelu(acc[mb][t][3]));
            if (mb & 1) {
                out[t][mb >> 1].z = lo;
                out[t][mb >> 1].w = hi;
            } else {
                out[t][mb >> 1].x = lo;
                out[t][mb >> 1].y = hi;
            }
        }
}

// Bulk trilinear velocity and void fraction at a particle from the packed
// features (fgrid[2c] = (eps_c, U_c)): u_bulk = sum_c w_pc U_c and
// eps_p = sum_c w_pc eps_c with the deposition weights (CIC or NGP).  Where the
// particle solid fraction exceeds phi_fp64 the sum is taken in FP64 (eps_c =
// 1 - phi_c is exact for phi_c >= 1/2, where it matters).
struct BulkCorners {
    Axis<float> x, y, z;
    float4 c[8];   // corner x + 2 y + 4 z of the stencil
};
__device__ __forceinline__ BulkCorners load_bulk_corners(const StepArgs<float> &a, const float4 &q) {
    const Geo<float> &g = a.g;
    BulkCorners b;
    b.x = cic_axis(q.x, g.sb[0], g.nb[0]);
    b.y = cic_axis(q.y, g.sb[1], g.nb[1]);
    b.z = cic_axis(q.z, g.sb[2], g.nb[2]);
    const int64_t nx = g.nb[0], nxy = (int64_t)g.nb[0] * g.nb[1];
    const int64_t z[2] = {b.z.lo * nxy, b.z.hi * nxy}, y[2] = {b.y.lo * nx, b.y.hi * nx};
#pragma unroll
    for (int k = 0; k < 8; ++k) b.c[k] = a.fgrid[2 * (z[k >> 2] + y[(k >> 1) & 1] + ((k & 1) ? b.x.hi : b.x.lo))];
    return b;
}
__device__ __forceinline__ float4 bulk_sample_packed(const StepArgs<float> &a, const float4 &q, const BulkCorners &b) {
    const Geo<float> &g = a.g;
    const Axis<float> &bx = b.x, &by = b.y, &bz = b.z;
    const int64_t nx = g.nb[0], nxy = (int64_t)g.nb[0] * g.nb[1];
    const float4 &c000 = b.c[0], &c001 = b.c[1], &c010 = b.c[2], &c011 = b.c[3], &c100 = b.c[4], &c101 = b.c[5],
                 &c110 = b.c[6], &c111 = b.c[7];
    const float sx = 1.f - bx.t, sy = 1.f - by.t, sz = 1.f - bz.t;
    auto tri = [&](float v000, float v001, float v010, float v011, float v100, float v101, float v110, float v111) {
        return sz * (sy * (sx * v000 + bx.t * v001) + by.t * (sx * v010 + bx.t * v011)) +
               bz.t * (sy * (sx * v100 + bx.t * v101) + by.t * (sx * v110 + bx.t * v111));
    };
    float4 r;
    r.x = tri(c000.y, c001.y, c010.y, c011.y, c100.y, c101.y, c110.y, c111.y);
    r.y = tri(c000.z, c001.z, c010.z, c011.z, c100.z, c101.z, c110.z, c111.z);
    r.z = tri(c000.w, c001.w, c010.w, c011.w, c100.w, c101.w, c110.w, c111.w);
    if (a.cic) {
        const float e = tri(c000.x, c001.x, c010.x, c011.x, c100.x, c101.x, c110.x, c111.x);
        if (1.f - e > a.phi_fp64) {
            const double gx = (double)q.x * (double)g.sb[0] - 0.5, gy = (double)q.y * (double)g.sb[1] - 0.5,
                         gz = (double)q.z * (double)g.sb[2] - 0.5;
            const double tx = gx - floor(gx), ty = gy - floor(gy), tz = gz - floor(gz);
            const double ux = 1.0 - tx, uy = 1.0 - ty, uz = 1.0 - tz;
            r.w = (float)(uz * (uy * (ux * (double)c000.x + tx * (double)c001.x) +
                                ty * (ux * (double)c010.x + tx * (double)c011.x)) +
                          tz * (uy * (ux * (double)c100.x + tx * (double)c101.x) +
                                ty * (ux * (double)c110.x + tx * (double)c111.x)));
        } else {
            r.w = e;
        }
    } else {
        const int ix = cell_axis(q.x, g.sb[0], g.nb[0]), iy = cell_axis(q.y, g.sb[1], g.nb[1]),
                  iz = cell_axis(q.z, g.sb[2], g.nb[2]);
        r.w = a.fgrid[2 * (ix + nx * iy + nxy * iz)].x;
    }
    return r;
}

// The stencil cells of one particle that lane group g gathers (unit 4 kb + g of
// its containing cell c0), and the centre cell.
struct StencilCells {
    float4 B0[7], B1[7], A0, A1;
    int ix, iy, iz;
};
__device__ __forceinline__ StencilCells load_stencil(const StepArgs<float> &a, int64_t c0, int g) {
    const Geo<float> &geo = a.g;
    const int64_t nx = geo.nb[0], nxy = (int64_t)geo.nb[0] * geo.nb[1];
    if (c0 < 0 || c0 >= geo.ncell) c0 = 0;
    StencilCells s;
    decode_cell(c0, geo.nb, s.ix, s.iy, s.iz);
#pragma unroll
    for (int kb = 0; kb < 7; ++kb) {
        const int u = 4 * kb + g;
        const int uu = u < 27 ? u : 13;
        const int dx = uu % 3 - 1, dy = (uu / 3) % 3 - 1, dz = uu / 9 - 1;
        const int64_t c = clampi(s.ix + dx, geo.nb[0]) + nx * clampi(s.iy + dy, geo.nb[1]) + nxy * clampi(s.iz + dz, geo.nb[2]);
        s.B0[kb] = a.fgrid[2 * c];
        s.B1[kb] = a.fgrid[2 * c + 1];
    }
    s.A0 = a.fgrid[2 * c0];
    s.A1 = a.fgrid[2 * c0 + 1];
    return s;
}

// Layer-1 slots 8 (4 kb + g) .. + 7 of one particle (clamped position and diameter
// q), standardised: a stencil cell's seven values, or the offsets and diameter
// (unit 27); the padding slots come out 0.
__device__ __forceinline__ uint4 stencil_slots(const StepArgs<float> &a, const float4 &q, const StencilCells &s, int kb,
                                               int g, const float (&mean)[8], const float (&inv)[8]) {
    const Geo<float> &geo = a.g;
    const bool off = kb == 6 && g == 3, centre = 4 * kb + g == 13;   // units 27 and 13
    const float4 &A0 = s.A0, &A1 = s.A1, &B0 = s.B0[kb], &B1 = s.B1[kb];
    float v[8] = {centre ? A0.x : B0.x - A0.x, centre ? A0.y : B0.y - A0.y, centre ? A0.z : B0.z - A0.z,
                  centre ? A0.w : B0.w - A0.w, centre ? A1.x : B1.x - A1.x, centre ? A1.y : B1.y - A1.y,
                  centre ? A1.z : B1.z - A1.z, 0.f};
    if (kb == 6) {
        const float o[4] = {q.x * geo.sb[0] - (float)s.ix, q.y * geo.sb[1] - (float)s.iy, q.z * geo.sb[2] - (float)s.iz,
                            q.w * geo.sb[0]};
#pragma unroll
        for (int i = 0; i < 8; ++i) v[i] = off ? (i < 4 ? o[i] : 0.f) : v[i];
    }
    float xs[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) xs[i] = (v[i] - mean[i]) * inv[i];
    return make_uint4(pack2(xs[0], xs[1]), pack2(xs[2], xs[3]), pack2(xs[4], xs[5]), pack2(xs[6], xs[7]));
}

// Persistent: each workgroup takes one contiguous range of the sorted particles
// (neighbouring cells: the stencil loads hit L1/L2), each wave kInfRows particles
// per round.  Lane (n, g) gathers, for tile t and slot group kb, unit 4 kb + g of
// particle 16 t + n; lanes with g < kInfTiles then finish particle 16 g + n:
// u = u_bulk + s * y and eps_p (both from the packed features), written to
// uf4[id].  With two waves per SIMD it is bound by the memory round trips of a
// round and by the standardisation's VALU work, not by the products: with a tile's
// loads after the other's conversion, the bulk corners loaded under a branch, and
// mean and 1/std read from LDS per feature under a condition (a branch each) it
// took 398 us for 1,250,000 particles; with all loads unconditional and in two and a
// half trips, and the tables in slot order (16-byte reads, no conditions), 314 us.
__global__ __launch_bounds__(kInfWaves * kWave) void k_infer(StepArgs<float> a) {
    __shared__ InferLds L;
    constexpr int NT = kInfTiles;
    const int lane = lane_id(), n = lane & 15, g = lane >> 4, wave = threadIdx.x >> 6;
    const MlpNet &net = a.net;
    // weights into LDS from the copies in slot order
    constexpr int kThreads = kInfWaves * kWave;
    stage_weights<7, 8, kThreads>(net.wtp[0], L.frag);
    stage_weights<4, 8, kThreads>(net.wtp[1], L.frag + kFrag1);
    stage_weights<4, 8, kThreads>(net.wtp[2], L.frag + kFrag1 + kFragH);
    stage_weights<4, 1, kThreads>(net.wtp[3], L.frag + kFrag1 + 2 * kFragH);
    for (int e = threadIdx.x; e < 3 * kHid + 16; e += kInfWaves * kWave) {
        const int l = e / kHid, m = e % kHid;
        constexpr int64_t kB0 = off_b(0), kB1 = off_b(1), kB2 = off_b(2), kB3 = off_b(3);
        const int64_t ob = l == 0 ? kB0 : (l == 1 ? kB1 : kB2);
        L.bias[e] = (l < 3) ? net.params[ob + m] : (m < kOut ? net.params[kB3 + m] : 0.f);
    }
    for (int e = threadIdx.x; e < kK1; e += kInfWaves * kWave) {
        const int u = e >> 3, i = e & 7;
        const int k = u < 27 ? (i < 7 ? 7 * u + i : -1) : (i < 4 ? 189 + i : -1);   // slot_of_feature(k) == e
        L.mean[e] = k >= 0 ? net.mean_inv[k] : 0.f;
        L.inv[e] = k >= 0 ? net.mean_inv[kK1 + k] : 0.f;
    }
    __syncthreads();

    const int64_t per = ((a.n + gridDim.x - 1) / gridDim.x + kInfRows - 1) / kInfRows * kInfRows;
    const int64_t s_begin = (int64_t)blockIdx.x * per;
    const int64_t s_end = (s_begin + per < a.n) ? s_begin + per : a.n;
    for (int64_t base = s_begin + (int64_t)wave * kInfRows; base < s_end; base += kInfWaves * kInfRows) {
        wave_sync();   // keeps the compiler from holding LDS rows in registers across rounds
        // Two memory round trips and part of a third: the particles; the stencil
        // cells of both tiles; then, while the second tile's are converted, the bulk
        // corners of the particle this lane finishes (tile g).  The lanes with none
        // and those past the end take another particle's, so that no load is
        // conditional.
        float4 q[NT];
        int64_t c[NT];
#pragma unroll
        for (int t = 0; t < NT; ++t) {
            int64_t s = base + 16 * t + n;
            s = s < s_end ? s : base;
            q[t] = a.sp[s];
            c[t] = a.keys[s];
        }
        const int64_t so = base + 16 * g + n;
        const bool own = (g < NT) && so < s_end;
        int64_t p = a.perm[own ? so : base];
        __builtin_amdgcn_sched_barrier(0);
        if (p < 0 || p >= a.n) p = 0;
        float4 qo = q[0];
#pragma unroll
        for (int t = 1; t < NT; ++t) {
            qo.x = g == t ? q[t].x : qo.x;
            qo.y = g == t ? q[t].y : qo.y;
            qo.z = g == t ? q[t].z : qo.z;
        }
        StencilCells sc[NT];
#pragma unroll
        for (int t = 0; t < NT; ++t) sc[t] = load_stencil(a, c[t], g);
        __builtin_amdgcn_sched_barrier(0);
        BulkCorners bc;
        uint4 x[NT][7];
#pragma unroll
        for (int t = 0; t < NT; ++t) {
#pragma unroll
            for (int kb = 0; kb < 7; ++kb) {
                const float4 *tm = reinterpret_cast<const float4 *>(L.mean + 8 * (4 * kb + g)),
                             *ti = reinterpret_cast<const float4 *>(L.inv + 8 * (4 * kb + g));
                const float4 m0 = tm[0], m1 = tm[1], i0 = ti[0], i1 = ti[1];
                const float mean[8] = {m0.x, m0.y, m0.z, m0.w, m1.x, m1.y, m1.z, m1.w};
                const float inv[8] = {i0.x, i0.y, i0.z, i0.w, i1.x, i1.y, i1.z, i1.w};
                x[t][kb] = stencil_slots(a, q[t], sc[t], kb, g, mean, inv);
                // (materialised here: the compiler would move the conversion past the
                // branches of bulk_sample_packed and keep all cells, spilling)
                asm volatile("" : "+v"(x[t][kb].x), "+v"(x[t][kb].y), "+v"(x[t][kb].z), "+v"(x[t][kb].w));
                __builtin_amdgcn_sched_barrier(0);   // a block at a time: the cells go as the operand comes
            }
            if (t == 0) {   // into the registers that the first tile's cells held
                bc = load_bulk_corners(a, qo);
                __builtin_amdgcn_sched_barrier(0);
            }
        }
        float4 r = bulk_sample_packed(a, qo, bc);
        uint4 h1[NT][4], h2[NT][4];
        chain_layer<NT, 7>(L, 0, L.bias, x, h1, lane, g);
        chain_layer<NT, 4>(L, kFrag1, L.bias + kHid, h1, h2, lane, g);
        chain_layer<NT, 4>(L, kFrag1 + kFragH, L.bias + 2 * kHid, h2, h1, lane, g);
        f32x4 y[NT];
        const f32x4 b4 = {L.bias[3 * kHid], L.bias[3 * kHid + 1], L.bias[3 * kHid + 2], 0.f};
#pragma unroll
        for (int t = 0; t < NT; ++t) y[t] = b4;
#pragma unroll
        for (int kb = 0; kb < 4; ++kb) {
            const bf16x8 w = as_bf16x8(L.frag[kFrag1 + 2 * kFragH + kb][lane]);
#pragma unroll
            for (int t = 0; t < NT; ++t) y[t] = mma(w, as_bf16x8(h1[t][kb]), y[t]);
        }
        // lane (n, 0) holds the 3 outputs of particle 16 t + n in y[t]
        float yo[3] = {0.f, 0.f, 0.f};
#pragma unroll
        for (int t = 0; t < NT; ++t)
#pragma unroll
            for (int j = 0; j < 3; ++j) {
                const float v = __shfl(y[t][j], n, kWave);
                if (t == g) yo[j] = v;
            }
        if (own) {
            r.x += net.scale[0] * yo[0];
            r.y += net.scale[1] * yo[1];
            r.z += net.scale[2] * yo[2];
            a.uf4[p] = r;
        }
    }
}

// Bricks of 8x8x8 bulk cells, one workgroup each.  The checked sample is every
// particle with id mod period = step mod period; where its relative L2 error
// against the fine lookup exceeds tol, every particle of the brick takes the
// fine lookup.  The brick's 64 (z, y) rows are one lane each: their sorted
// ranges are loaded at once and prefix-summed across the wave (by every wave),
// and the brick's particles are then processed 256 at a time in that flattened
// order.  Bound by the chain of dependent loads (id, sampled particle, fine
// nodes): a dense brick's 3,400 particles took one wave 13 rounds, 118 us for
// 1024 bricks.  Per workgroup: fallback count, sampled squared error and
// reference, sample count (FP64 partials, fixed order).
constexpr int kBrick = 8;

__global__ __launch_bounds__(kBlock) void k_check(StepArgs<float> a) {
    static_assert(kBrick * kBrick == kWave, "one lane per (z, y) row of a brick");
    __shared__ double red[kWavesPerBlock];
    __shared__ int32_t pre[kWave + 1];   // particles before each row (exclusive prefix)
    __shared__ int64_t row0[kWave];      // first sorted position of each row
    const int lane = lane_id(), wave = threadIdx.x >> 6;
    const int64_t brick = blockIdx.x;
    const Geo<float> &geo = a.g;
    const int bx = (geo.nb[0] + kBrick - 1) / kBrick, by = (geo.nb[1] + kBrick - 1) / kBrick;
    const int ox = (int)(brick % bx) * kBrick, oy = (int)((brick / bx) % by) * kBrick,
              oz = (int)(brick / ((int64_t)bx * by)) * kBrick;
    const int wx = (ox + kBrick < geo.nb[0]) ? kBrick : geo.nb[0] - ox;
    // lane r owns row (dz, dy) = (r / 8, r % 8): its particles are the
    // contiguous sorted range of cells ox .. ox + wx - 1 of that row
    const int dz = lane / kBrick, dy = lane % kBrick;
    int64_t s0 = 0, s1 = 0;
    if (oz + dz < geo.nb[2] && oy + dy < geo.nb[1]) {
        const int64_t c0 = ox + (int64_t)geo.nb[0] * ((oy + dy) + (int64_t)geo.nb[1] * (oz + dz));
        s0 = seg_clamp(a.start[c0], a.n);
        s1 = seg_clamp(a.start[c0 + wx], a.n);
    }
    int32_t incl = (int32_t)(s1 - s0);   // inclusive prefix over the lanes (rows in order)
#pragma unroll
    for (int o = 1; o < kWave; o <<= 1) {
        const int32_t v = __shfl_up(incl, o, kWave);
        if (lane >= o) incl += v;
    }
    const int32_t total = __shfl(incl, kWave - 1, kWave);
    if (wave == 0) {
        pre[lane + 1] = incl;
        if (lane == 0) pre[0] = 0;
        row0[lane] = s0;
    }
    __syncthreads();
    // flattened index j -> row (last r with pre[r] <= j) -> sorted position
    auto position = [&](int32_t j) {
        int lo = 0, hi = kWave;   // pre[lo] <= j < pre[hi]
        while (hi - lo > 1) {
            const int mid = (lo + hi) >> 1;
            if (pre[mid] <= j) lo = mid;
            else hi = mid;
        }
        return row0[lo] + (j - pre[lo]);
    };
    const int64_t period = a.mlp_period, phase = ((a.step % period) + period) % period;
    double err = 0.0, ref = 0.0, ns = 0.0, nfall = 0.0;
    // kU particles of a thread per round: their ids are loaded together (one
    // round trip instead of kU), then taken in the thread's order j
    constexpr int kU = 4;
    for (int32_t j0 = threadIdx.x; j0 < total; j0 += kU * kBlock) {
        int64_t s[kU], p[kU];
#pragma unroll
        for (int u = 0; u < kU; ++u) {
            const int32_t j = j0 + u * kBlock;
            s[u] = position(j < total ? j : j0);
            p[u] = a.perm[s[u]];
        }
#pragma unroll
        for (int u = 0; u < kU; ++u) {
            if (j0 + u * kBlock >= total) break;
            int64_t pu = p[u];
            if (pu < 0 || pu >= a.n) pu = 0;
            if (pu % period != phase) continue;
            float ux, uy, uz;
            fine_velocity(a.sp[s[u]], a, ux, uy, uz);
            const float4 m = a.uf4[pu];
            const double ex = (double)m.x - ux, ey = (double)m.y - uy, ez = (double)m.z - uz;
            err += ex * ex + ey * ey + ez * ez;
            ref += (double)ux * ux + (double)uy * uy + (double)uz * uz;
            ns += 1.0;
        }
    }
    const double terr = block_sum(err, red), tref = block_sum(ref, red), tns = block_sum(ns, red);
    const double tol = (double)a.mlp_tol;
    if (tns > 0.0 && terr > tol * tol * tref) {   // uniform over the workgroup
        for (int32_t j = threadIdx.x; j < total; j += kBlock) {
            const int64_t s = position(j);
            int64_t p = a.perm[s];
            if (p < 0 || p >= a.n) p = 0;
            float4 m = a.uf4[p];
            fine_velocity(a.sp[s], a, m.x, m.y, m.z);
            a.uf4[p] = m;
            nfall += 1.0;
        }
    }
    const double tfall = block_sum(nfall, red);
    if (threadIdx.x == 0) {
        const double vals[4] = {tfall, terr, tref, tns};
        const int slots[4] = {SL_NFALL, SL_MLPERR, SL_MLPREF, SL_MLPSAMP};
        for (int k = 0; k < 4; ++k) a.part[slots[k] * a.part_stride + blockIdx.x] = vals[k];
    }
}

}  // namespace mlp

// ---------------------------------------------------------------------------
// Host launchers
// ---------------------------------------------------------------------------
int64_t bricks_of(const int nb[3]) {
    int64_t b = 1;
    for (int a = 0; a < 3; ++a) b *= (nb[a] + mlp::kBrick - 1) / mlp::kBrick;
    return b;
}
int64_t mlp_check_blocks(int64_t n_bricks) { return n_bricks; }

// Workgroups of a persistent kernel: one per compute unit, or fewer.
static unsigned persistent_grid(int64_t items) {
    int dev = 0, ncu = 256;
    if (hipGetDevice(&dev) == hipSuccess) (void)hipDeviceGetAttribute(&ncu, hipDeviceAttributeMultiprocessorCount, dev);
    if (ncu < 1) ncu = 1;
    return (unsigned)(items < ncu ? (items > 0 ? items : 1) : ncu);
}

void launch_mlp_pack(const StepArgs<float> &a, hipStream_t st) {
    hipLaunchKernelGGL(mlp::k_pack, dim3((unsigned)((a.g.ncell + kBlock - 1) / kBlock)), dim3(kBlock), 0, st, a);
}

void launch_mlp_infer(const StepArgs<float> &a, hipStream_t st) {
    if (a.n <= 0) return;
    const int64_t rounds = (a.n + mlp::kInfRows - 1) / mlp::kInfRows;
    hipLaunchKernelGGL(mlp::k_infer, dim3(persistent_grid((rounds + mlp::kInfWaves - 1) / mlp::kInfWaves)),
                       dim3(mlp::kInfWaves * kWave), 0, st, a);
}

void launch_mlp_check(const StepArgs<float> &a, hipStream_t st) {
    hipLaunchKernelGGL(mlp::k_check, dim3((unsigned)mlp_check_blocks(a.n_bricks)), dim3(kBlock), 0, st, a);
}

namespace mlp {

static WPtrs wptrs(const NetBufs &net) {
    WPtrs w;
    for (int l = 0; l < 4; ++l) {
        w.wt[l] = net.wt[l];
        w.wn[l] = net.wn[l];
        w.wtp[l] = net.wtp[l];
        w.wnp[l] = net.wnp[l];
    }
    return w;
}

static unsigned blocks(int64_t n) { return (unsigned)((n + kBlock - 1) / kBlock); }

hipError_t launch_cast(const NetBufs &net, hipStream_t st) {
    hipLaunchKernelGGL(k_cast, dim3(blocks(kNParam)), dim3(kBlock), 0, st, net.params, wptrs(net));
    return hipGetLastError();
}

hipError_t launch_adam(const NetBufs &net, const float *grads, float lr, float b1, float omb1, float b2, float omb2,
                       float eps, float c1, float c2, hipStream_t st) {
    hipLaunchKernelGGL(k_adam, dim3(blocks(kNParam)), dim3(kBlock), 0, st, grads, net.params, net.m, net.v, wptrs(net),
                       lr, b1, omb1, b2, omb2, eps, c1, c2);
    return hipGetLastError();
}

hipError_t launch_forward(const NetBufs &net, const float *feat, int64_t B, float *y, hipStream_t st) {
    if (B <= 0) return hipSuccess;
    ForwardNet fn;
    for (int l = 0; l < 4; ++l) fn.wt[l] = net.wt[l];
    fn.params = net.params;
    fn.mean_inv = net.mean_inv;
    hipLaunchKernelGGL(k_forward, dim3(persistent_grid((B + kFwdRows - 1) / kFwdRows)), dim3(kFwdWaves * kWave), 0, st,
                       feat, B, fn, y);
    return hipGetLastError();
}

hipError_t launch_gradients(const NetBufs &net, const TrainBufs &tb, const float *feat, const float *resid,
                            const int32_t *idx, int64_t nrows, int64_t B, const float inv_scale[3], float *grads,
                            float *loss, hipStream_t st) {
    TrainArgs a;
    a.feat = feat;
    a.resid = resid;
    a.idx = idx;
    a.nrows = nrows;
    a.B = B;
    a.mean_inv = net.mean_inv;
    for (int j = 0; j < 3; ++j) a.is[j] = inv_scale[j];
    a.inv_b = (float)(1.0 / (double)B);
    a.params = net.params;
    a.wt0 = net.wt[0];
    for (int l = 0; l < 4; ++l) {
        a.wtp[l] = net.wtp[l];
        a.wnp[l] = net.wnp[l];
        a.part_b[l] = tb.part_b[l];
    }
    a.tr = tb.tr;
    a.loss_part = tb.loss_part;
    if (B <= 0 || B % kTrainGroupRows != 0) return hipErrorInvalidValue;   // every workgroup has both tiles
    const unsigned nt = (unsigned)n_train_groups(B);
    hipLaunchKernelGGL(k_train_tile, dim3(nt), dim3(kTrainThreads), 0, st, a);
    const unsigned nc = (unsigned)n_chunks(B);
    const dim3 bw(kWgradWaves * kWave);
    WgradParts wp;
    for (int l = 0; l < 4; ++l) wp.w[l] = tb.part_w[l];
    hipLaunchKernelGGL(k_wgrad, dim3(nc, 2), bw, 0, st, tb.tr, B, wp);
    GradParts parts;
    for (int l = 0; l < 4; ++l) {
        parts.w[l] = tb.part_w[l];
        parts.b[l] = tb.part_b[l];
    }
    hipLaunchKernelGGL(k_reduce, dim3(kRedWBlocks + kRedBBlocks + (loss ? 1 : 0)), dim3(kRedThreads), 0, st, parts,
                       (int64_t)nc, (int64_t)nt, grads, tb.loss_part, B / 16, loss);
    return hipGetLastError();
}

hipError_t launch_column_stats(const float *x, int64_t n, int cols, double *part, int64_t nchunk, double *mean,
                               double *std, hipStream_t st) {
    const int64_t rows_per = (n + nchunk - 1) / nchunk;
    hipLaunchKernelGGL(k_colsum, dim3((unsigned)nchunk), dim3(kBlock), 0, st, x, n, cols, rows_per, nullptr, part);
    hipLaunchKernelGGL(k_colfinish, dim3(1), dim3(kBlock), 0, st, part, nchunk, cols, n, 0, mean);
    hipLaunchKernelGGL(k_colsum, dim3((unsigned)nchunk), dim3(kBlock), 0, st, x, n, cols, rows_per, mean, part);
    hipLaunchKernelGGL(k_colfinish, dim3(1), dim3(kBlock), 0, st, part, nchunk, cols, n, 1, std);
    return hipGetLastError();
}

hipError_t launch_features(const int nb[3], const double box[3], int64_t n, const float *pos, const float *diam,
                           const float *phi, const float *U, const float *G, const float *u_fine,
                           const int32_t *sel, int64_t nsel, float *feat, float *u_bulk, float *resid,
                           hipStream_t st) {
    if (nsel <= 0) return hipSuccess;
    Geo<float> g;
    for (int a = 0; a < 3; ++a) {
        g.nb[a] = nb[a];
        g.nf[a] = nb[a];
        g.L[a] = (float)box[a];
        g.sb[a] = (float)((double)nb[a] / box[a]);
        g.sf[a] = g.sb[a];
        g.hb[a] = (float)(box[a] / (double)nb[a]);
    }
    g.ncell = (int64_t)nb[0] * nb[1] * nb[2];
    g.nfine = g.ncell;
    g.vb = (box[0] / nb[0]) * (box[1] / nb[1]) * (box[2] / nb[2]);
    g.vf = g.vb;
    g.inv_vb = (float)(1.0 / g.vb);
    hipLaunchKernelGGL(k_features, dim3(blocks(nsel)), dim3(kBlock), 0, st, g, n, pos, diam, phi, U, G, u_fine, sel, nsel,
                       feat, u_bulk, resid);
    return hipGetLastError();
}

}  // namespace mlp
}  // namespace cpl
