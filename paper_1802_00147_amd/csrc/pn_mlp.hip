// pn_mlp.hip -- learned surrogate of the FLI scan: a 7-256-256-256-2 ReLU
// multilayer perceptron trained and evaluated on gfx950 matrix cores.
//
// General products run in one hand-written kernel, k_gemm_bf16: bfloat16
// operands, FP32 accumulation on v_mfma_f32_16x16x32_bf16, 64x64 output tiles
// per 256-thread workgroup (each wavefront a 32x32 quarter as 2x2 MFMA
// tiles), operands staged through LDS with K contiguous so that a lane reads
// its eight K values with one 16-byte LDS load, and fused epilogues (bias as
// the accumulators' start, ReLU, ReLU-mask of the backward pass, FP32 and/or
// bfloat16 stores).  Arbitrary strides let the same kernel form X W^T, G W
// and G^T H.  A training step is two kernels: k_mlp_train (forward pass, loss,
// layer gradients) and k_mlp_update (weight and bias gradients, Adam).
// Inference over scan grids is one persistent kernel, k_mlp_infer.  All take
// their products with the same arithmetic as k_gemm_bf16.  The
// surrogate-assisted scan (pn_surrogate_scan) strings these together with
// the FP64 scans.
#include <hip/hip_runtime.h>

#include <cmath>
#include <cstdint>
#include <cstdio>
#include <cstring>
#include <algorithm>
#include <type_traits>
#include <vector>

#include "pn.h"

typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 bf16x8;
typedef __attribute__((__vector_size__(4 * sizeof(float)))) float f32x4;

namespace pn_detail {
void set_last_error(const char* what, const char* msg);   // pn_kernels.hip
}

namespace {

constexpr int BM = 64, BN = 64, BK = 32, LDSK = BK + 8;
constexpr int kIn[4] = {7, 256, 256, 256};
constexpr int kOut[4] = {256, 256, 256, 2};
constexpr int kFeatLd = 8;     // feature rows are padded to 8 values


// FP32 -> bfloat16, round to nearest even (one v_cvt_pk_bf16_f32 on gfx950).
__device__ __forceinline__ uint16_t f2bf(float f) { return __builtin_bit_cast(uint16_t, (__bf16)f); }

__device__ __forceinline__ float bf2f(uint16_t b) { return __uint_as_float(((uint32_t)b) << 16); }

// ReLU applied after the rounding to bfloat16: a value with its sign bit set
// (negative, or -0) becomes +0, any other stays.  For finite values this is
// the rounding of max(x, 0); on a packed pair it is one signed 16-bit max
// against zero (v_pk_max_i16).
typedef short short2v __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x2v __attribute__((ext_vector_type(2)));
typedef float float2v __attribute__((ext_vector_type(2)));
__device__ __forceinline__ uint16_t relu_bf16(uint16_t b) { return (b & 0x8000u) ? (uint16_t)0 : b; }
// Two FP32 values to a packed bfloat16 pair (a low), each rounded as f2bf.
__device__ __forceinline__ uint32_t pack_bf16x2(float a, float b) {
    return __builtin_bit_cast(uint32_t, __builtin_convertvector((float2v){a, b}, bf16x2v));
}
__device__ __forceinline__ uint32_t relu_bf16x2(uint32_t p) {
    const short2v v = __builtin_bit_cast(short2v, p);
    return __builtin_bit_cast(uint32_t, __builtin_elementwise_max(v, short2v{0, 0}));
}

struct GemmArgs {
    int M, N, K;
    const uint16_t* A;
    int64_t sam, sak;          // A(m, k) = A[m * sam + k * sak]
    const uint16_t* B;
    int64_t sbk, sbn;          // B(k, n) = B[k * sbk + n * sbn]
    const float* bias;         // [N] or null
    const uint16_t* mask;      // ReLU mask source [M x N] (value > 0 keeps), or null
    int64_t ldm;
    float* Cf;                 // FP32 result or null
    int64_t ldcf;
    uint16_t* Cb;              // bfloat16 result or null
    int64_t ldcb;
    int relu;
    int amode, bmode;          // operand staging: 0 element-wise, 1 K contiguous, 2 M (N) contiguous
};

// Staging modes of an operand whose element (r, k) -- r the row of the
// output tile (m for A, n for B) -- sits at p[r * sr + k * sk]:
//   1: K contiguous (sk = 1, sr a multiple of 8, 16-byte aligned base):
//      one 16-byte load of 8 K values per thread;
//   2: r contiguous (sr = 1, sk a multiple of 8, aligned): one 16-byte load
//      of 8 rows at one K per thread, transposed into LDS;
//   0: element by element.
int stage_mode(const uint16_t* p, int64_t sr, int64_t sk) {
    const bool aligned = (reinterpret_cast<uintptr_t>(p) & 15u) == 0;
    if (aligned && sk == 1 && sr % 8 == 0) return 1;
    if (aligned && sr == 1 && sk % 8 == 0) return 2;
    return 0;
}

// K slices staged in LDS between two barriers: their global loads are all
// in flight before the first LDS store, so a K range of 256 waits for memory
// twice instead of eight times.
constexpr int kStageSlices = 4;

// One 16-byte chunk of a tile: this thread's part of slice (r0.., k0..) of
// the operand whose element (r, k) sits at p[r * sr + k * sk], zero outside
// [0, R) x [0, K).  Mode 1 gives 8 K values of one row (row tid / 4, K offset
// 8 (tid % 4)); mode 2 gives 8 rows at one K (K offset tid / 8, rows
// 8 (tid % 8) ..); see stage_mode.
__device__ __forceinline__ uint4 load_chunk(const uint16_t* p, int64_t sr, int64_t sk, int mode, int64_t r0,
                                            int64_t R, int64_t k0, int64_t K, int tid) {
    union { uint4 v; uint16_t e[8]; } u;
    if (mode == 1) {
        const int64_t row = r0 + (tid >> 2), k = k0 + (tid & 3) * 8;
        if (row < R && k + 8 <= K) {
            u.v = *reinterpret_cast<const uint4*>(p + row * sr + k);
        } else {
#pragma unroll
            for (int t = 0; t < 8; ++t) u.e[t] = (row < R && k + t < K) ? p[row * sr + (k + t)] : (uint16_t)0;
        }
    } else {
        const int64_t k = k0 + (tid >> 3), row = r0 + (tid & 7) * 8;
        if (k < K && row + 8 <= R) {
            u.v = *reinterpret_cast<const uint4*>(p + row + k * sk);
        } else {
#pragma unroll
            for (int t = 0; t < 8; ++t) u.e[t] = (k < K && row + t < R) ? p[(row + t) + k * sk] : (uint16_t)0;
        }
    }
    return u.v;
}

// Writes a chunk from load_chunk into tile[64][LDSK] (mode 2 transposes it).
__device__ __forceinline__ void store_chunk(uint16_t (*tile)[LDSK], uint4 v, int mode, int tid) {
    if (mode == 1) {
        *reinterpret_cast<uint4*>(&tile[tid >> 2][(tid & 3) * 8]) = v;
    } else {
        union { uint4 v; uint16_t e[8]; } u;
        u.v = v;
        const int c = tid >> 3, r = (tid & 7) * 8;
#pragma unroll
        for (int t = 0; t < 8; ++t) tile[r + t][c] = u.e[t];
    }
}

// Fill tiles[s][64][LDSK], s < ns, with element (r0 + r, k0 + s BK + c) of
// the operand (row r, K offset c), zero outside [0, R) x [0, K).
__device__ __forceinline__ void stage_tiles(uint16_t (*tiles)[BM][LDSK], int ns, const uint16_t* p, int64_t sr,
                                            int64_t sk, int mode, int64_t r0, int64_t R, int64_t k0, int64_t K,
                                            int tid) {
    if (mode == 0) {
        for (int s = 0; s < ns; ++s)
            for (int e = tid; e < 64 * BK; e += 256) {
                const int r = e / BK, c = e % BK;
                const int64_t row = r0 + r, k = k0 + s * BK + c;
                tiles[s][r][c] = (row < R && k < K) ? p[row * sr + k * sk] : (uint16_t)0;
            }
        return;
    }
    if (ns == kStageSlices && r0 + BM <= R && k0 + kStageSlices * BK <= K) {
        // Whole tiles inside the operand (the same for every thread): the
        // loads go out back to back, with no bounds branch between them.
        const int64_t off = mode == 1 ? (r0 + (tid >> 2)) * sr + k0 + (tid & 3) * 8
                                      : r0 + (tid & 7) * 8 + (k0 + (tid >> 3)) * sk;
        const int64_t step = mode == 1 ? BK : BK * sk;
        uint4 v[kStageSlices];
#pragma unroll
        for (int s = 0; s < kStageSlices; ++s) v[s] = *reinterpret_cast<const uint4*>(p + off + s * step);
#pragma unroll
        for (int s = 0; s < kStageSlices; ++s) store_chunk(tiles[s], v[s], mode, tid);
        return;
    }
    for (int s = 0; s < ns; ++s) store_chunk(tiles[s], load_chunk(p, sr, sk, mode, r0, R, k0 + s * BK, K, tid), mode, tid);
}

// C = A B (+ bias) (ReLU) (* mask), M x N: grid (N / 64, M / 64), one 64 x 64
// output tile per workgroup, FP32 accumulation, staged through LDS
// (kStageSlices K slices each).  The MFMAs take the K slices in increasing
// order, one 16x16x32 step per slice and output block.
__global__ __launch_bounds__(256) void k_gemm_bf16(GemmArgs g) {
    __shared__ __attribute__((aligned(16))) uint16_t As[kStageSlices][BM][LDSK];
    __shared__ __attribute__((aligned(16))) uint16_t Bt[kStageSlices][BN][LDSK];
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
    const int64_t m0 = (int64_t)blockIdx.y * BM, n0 = (int64_t)blockIdx.x * BN;
    const int wm = (wave >> 1) * 32, wn = (wave & 1) * 32;
    const int lr = lane & 15, lk = (lane >> 4) * 8;
    // The bias is the accumulators' starting value: the MFMAs add the K slices
    // to it.
    f32x4 acc[2][2];
#pragma unroll
    for (int j = 0; j < 2; ++j) {
        const int64_t n = n0 + wn + 16 * j + lr;
        const float b0 = (g.bias && n < g.N) ? g.bias[n] : 0.0f;
#pragma unroll
        for (int i = 0; i < 2; ++i) acc[i][j] = f32x4{b0, b0, b0, b0};
    }
    for (int64_t k0 = 0; k0 < g.K; k0 += kStageSlices * BK) {
        const int64_t left = (g.K - k0 + BK - 1) / BK;
        const int ns = left < kStageSlices ? (int)left : kStageSlices;
        stage_tiles(As, ns, g.A, g.sam, g.sak, g.amode, m0, g.M, k0, g.K, tid);
        stage_tiles(Bt, ns, g.B, g.sbn, g.sbk, g.bmode, n0, g.N, k0, g.K, tid);
        __syncthreads();
#pragma unroll
        for (int s = 0; s < kStageSlices; ++s) {
            if (s < ns) {
                bf16x8 a[2], b[2];
#pragma unroll
                for (int i = 0; i < 2; ++i) a[i] = *reinterpret_cast<const bf16x8*>(&As[s][wm + 16 * i + lr][lk]);
#pragma unroll
                for (int j = 0; j < 2; ++j) b[j] = *reinterpret_cast<const bf16x8*>(&Bt[s][wn + 16 * j + lr][lk]);
#pragma unroll
                for (int i = 0; i < 2; ++i)
#pragma unroll
                    for (int j = 0; j < 2; ++j)
                        acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[i], b[j], acc[i][j], 0, 0, 0);
            }
        }
        __syncthreads();
    }
    // Accumulator layout: element v of lane l is row 4 (l / 16) + v, column l % 16.
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int64_t m = m0 + wm + 16 * i + (lane >> 4) * 4 + v;
                const int64_t n = n0 + wn + 16 * j + lr;
                if (m >= g.M || n >= g.N) continue;
                const float x = acc[i][j][v];
                const bool keep = !g.mask || bf2f(g.mask[m * g.ldm + n]) > 0.0f;
                if (g.Cf) g.Cf[m * g.ldcf + n] = keep ? (g.relu ? fmaxf(x, 0.0f) : x) : 0.0f;
                if (g.Cb) {
                    const uint16_t y = g.relu ? relu_bf16(f2bf(x)) : f2bf(x);
                    g.Cb[m * g.ldcb + n] = keep ? y : (uint16_t)0;
                }
            }
}

// Rows idx[b] (or b) of the FP32 features -> bfloat16 [rows x 8].
__global__ __launch_bounds__(256) void k_gather_rows(const float* feat, const int32_t* idx, int64_t rows,
                                                     int64_t row0, uint16_t* X) {
    const int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (e >= rows * kFeatLd) return;
    const int64_t b = e / kFeatLd;
    const int c = (int)(e % kFeatLd);
    const int64_t r = idx ? (int64_t)idx[b] : row0 + b;
    X[e] = c < 7 ? f2bf(feat[r * kFeatLd + c]) : (uint16_t)0;
}

constexpr int FLD = 256 + 8;        // LDS row stride of an activation buffer (elements)

__device__ __forceinline__ bf16x8 load_bf16x8(const uint16_t* p) {
    return *reinterpret_cast<const bf16x8*>(p);
}

// Fragment order of a 256 x 256 bfloat16 operand whose element (col, k) is the
// product's column col at depth k: the 16-byte piece of lane l for column
// block cb (16 columns) and K slice sl (32 deep) -- column 16 cb + l % 16, depths
// 32 sl + 8 (l / 16) .. + 8 -- is piece (cb * 8 + sl) * 64 + l, so a wavefront loads
// a fragment as 1 KB in a row.
// (cb is the same in all lanes of a wavefront: the address is a scalar base and
// one 32-bit lane offset.)
__device__ __forceinline__ bf16x8 load_frag(const uint16_t* F, int cb, int sl, int lane) {
    const char* base = reinterpret_cast<const char*>(F) + __builtin_amdgcn_readfirstlane(cb * 8 + sl) * 1024;
    return *reinterpret_cast<const bf16x8*>(base + (uint32_t)(lane * 16));
}

// What the training pass reads and leaves behind: rows idx[r] of the
// features; the gathered bfloat16 inputs x_out [n][8] and hidden activations
// h_out[l] [n][256] (16-byte aligned); the batch's mean loss added to *loss
// and its gradient with respect to the two outputs in gout [n][2]; the layer
// gradients g3 = (g4 W4) * (h3 > 0), g2 = (g3 W3) * (h2 > 0) and g1 = (g2 W2) * (h1 > 0)
// in g_out[2], [1], [0] [n][256] (all bfloat16).  The same tensors go out a
// second time in row-block order (Blocks).  Only that copy is read; the row-major
// one is what a step leaves for its caller, and without KEEP it is not written.
// out may be null.  Hidden weights come in fragment order: wf[0], wf[1] =
// W2, W3 (columns: outputs), wt[0], wt[1] = W2, W3 transposed (columns: inputs);
// W1 comes with its rows padded to eight values.
// A bfloat16 tensor of n rows and C columns in row-block order: element (r, c) of
// a slice of 32 rows at ((r / 8) C + c) 8 + r % 8, so that the eight rows which a
// lane of the weight gradients' products takes lie together.  The n / 32 whole
// slices lie one behind the other at `full`; the rest of the rows, if any, are a
// slice of their own at `last`, with zeros in the rows from n on.  (Eight whole
// rows take the same bytes in this order as in row-major order: `full` may be the
// place of the row-major tensor, in which the slice at `last` would not fit.)
struct Blocks {
    uint16_t* full;
    uint16_t* last;
};

struct TrainIO {
    const uint16_t* w0;              // layer 1 [256][8]
    const uint16_t* w3;              // layer 4 [2][256]
    const float* b[4];
    const uint16_t* wf[2];
    const uint16_t* wt[2];
    const float* feat;
    const float* label;
    const float* target;
    const int32_t* idx;
    int64_t n;
    float* out;
    float* loss;
    uint16_t* x_out;
    uint16_t* h_out[3];
    uint16_t* gout;
    uint16_t* g_out[3];
    Blocks xT, hT[3], g4T, gT[3];
};

constexpr int kTrainFT = 16;        // rows of a training tile

// Training pass of one step over the batch rows, in tiles of 16 rows (a
// batch of a few thousand rows spreads over a hundred or more workgroups).
// Wavefront w owns columns 32w .. 32w+31 of every layer (2 column blocks of
// 16); results are in the MFMA's own layout (element v of lane l is row
// 4 (l / 16) + v, column l % 16).  Products, K-slice order, bias-started
// accumulators and epilogues are those of k_gemm_bf16.
//
// A tile is a chain of seven small products, so the time is latency: of the
// weights (512 KB a workgroup, 64 B a clock: 8,200 cycles), of the gathered rows
// and of each stage.  Therefore
//  - fragments come in fragment order, W2 and W3 before the tile starts, and
//    W3^T and W2^T into the same registers once the forward product of that matrix
//    is through, a quarter at a time: a wavefront that asks for a whole operand at
//    once stands 2,000 cycles until its last load is taken;
//  - every wavefront forms the output layer and the loss gradient of all 16 rows
//    itself, one row per lane with both outputs (weights as the first operand),
//    so that the gradient is in place for g3's product without an exchange, and
//    the loss's value comes after everything that another wavefront waits for;
//  - ReLU masks stay in the lane that formed the activation.
// 25 us at 2,048 rows before (weights row-major, loss on one wavefront with
// a barrier on each side), 13.0 now (median of 57; 11.7 at the least), and 14.0 where
// the row-major copies are kept.  The wavefronts wait for memory or at barriers in
// 45% of their cycles, to issue in 32%, and an MFMA is in flight in 12%.
// APART: the last slice, not whole, is apart from the others.
template <bool KEEP, bool APART>
__global__ __launch_bounds__(512) void k_mlp_train(TrainIO io) {
    constexpr int FT = kTrainFT;
    __shared__ __attribute__((aligned(16))) uint16_t h1s[FT][FLD];
    __shared__ __attribute__((aligned(16))) uint16_t h2s[FT][FLD];   // later the g1 staging
    __shared__ __attribute__((aligned(16))) uint16_t h3s[FT][FLD];   // later g2
    __shared__ __attribute__((aligned(16))) uint16_t g3s[FT][FLD];
    __shared__ __attribute__((aligned(16))) uint16_t w4s[2][256];    // the output layer's weights
    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
    const int lr = lane & 15, lq = lane >> 4, lk = lq * 8;
    const int c0 = 32 * wave;                         // first column of this wavefront
    const int64_t n = io.n;
    const int64_t tile = blockIdx.x, ntiles = gridDim.x;
    const int64_t r0 = tile * FT;
    const bool part = APART && (r0 >> 5) >= (n >> 5); // the tile is in the slice at `last`
    // This tile's rows in a tensor of C columns in row-block order.
    auto rows_of = [&](const Blocks& t, int C) { return part ? t.last + (r0 & 31) * C : t.full + r0 * C; };
    const bool live = r0 + lr < n;                    // rows past n repeat row n - 1 and are never stored
    const int32_t src = io.idx[live ? r0 + lr : n - 1];
    const uint16_t w4v = io.w3[tid];                  // 512 threads, 2 x 256 weights

    bf16x8 wf[2][2][8];                               // two 256-deep operands of this wavefront's columns
    auto load_weights = [&](int slot, const uint16_t* F, int s0, int s1) {   // K slices [s0, s1)
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int sl = s0; sl < s1; ++sl)
#pragma unroll
            for (int j = 0; j < 2; ++j) wf[slot][j][sl] = load_frag(F, 2 * wave + j, sl, lane);
        __builtin_amdgcn_sched_barrier(0);
    };
    // Layer 1 fragments (K = 7; only the lanes of K-group 0 carry values).
    bf16x8 wf0[2];
#pragma unroll
    for (int j = 0; j < 2; ++j) {
        wf0[j] = bf16x8{};
        if (lq == 0) wf0[j] = load_bf16x8(io.w0 + (c0 + 16 * j + lr) * 8);
    }
    // Biases of this lane's columns, the accumulators' start.
    float bias[3][2];
#pragma unroll
    for (int l = 0; l < 3; ++l)
#pragma unroll
        for (int j = 0; j < 2; ++j) bias[l][j] = io.b[l][c0 + 16 * j + lr];
    const float b40 = io.b[3][0], b41 = io.b[3][1];
    // The row's index and W2 are on their way; then the features, label and
    // target of row lr (the lanes of K-groups 1-3 meet zero weights), W3 behind them.
    load_weights(0, io.wf[0], 0, 8);
    const float* fr = io.feat + (int64_t)src * kFeatLd;
    const float4 f0 = *reinterpret_cast<const float4*>(fr);
    const float4 f1 = *reinterpret_cast<const float4*>(fr + 4);
    const float lab = io.label[src], tgt = io.target[src];
    load_weights(1, io.wf[1], 0, 8);
    w4s[tid >> 8][tid & 255] = w4v;               // read after barriers

    // Rows 4 lq .. of this tile below n, of the four this lane's elements
    // belong to; pad: the tile also clears the 16 rows up to a multiple of 32.
    const int live4 = (int)(n - r0 < FT ? n - r0 : FT) - 4 * lq;
    const bool pad = (ntiles & 1) && tile == ntiles - 1;
    const int offT = (lq >> 1) * 4096 + lr * 16 + (lq & 1) * 8;

    f32x4 acc[2];
    uint32_t mask[3] = {0u, 0u, 0u};              // bit 4 j + v of layer l: its activation is positive
    // One tensor's columns of this wavefront: row-major through LDS (where
    // the next product reads it, too) and in row-block order.  The LDS
    // reads are of what this wavefront has just written, in order.
    auto put = [&](uint16_t (*h)[FLD], const uint16_t (&y)[2][4], uint16_t* dst, const Blocks& dstT) {
        char* T = reinterpret_cast<char*>(rows_of(dstT, 256) + c0 * 8);      // the same in all lanes
#pragma unroll
        for (int j = 0; j < 2; ++j) {
#pragma unroll
            for (int v = 0; v < 4; ++v) h[4 * lq + v][c0 + 16 * j + lr] = y[j][v];
            uint2 u;
            u.x = (0 < live4 ? (uint32_t)y[j][0] : 0u) | (1 < live4 ? (uint32_t)y[j][1] << 16 : 0u);
            u.y = (2 < live4 ? (uint32_t)y[j][2] : 0u) | (3 < live4 ? (uint32_t)y[j][3] << 16 : 0u);
            *reinterpret_cast<uint2*>(T + (uint32_t)(offT + 256 * j)) = u;
            if (pad) *reinterpret_cast<uint2*>(T + (uint32_t)(offT + 256 * j + 8192)) = make_uint2(0u, 0u);
        }
        if (!KEEP) return;
        __builtin_amdgcn_wave_barrier();
        const int r = lane >> 2;
        const uint4 q = *reinterpret_cast<const uint4*>(&h[r][c0 + 8 * (lane & 3)]);
        char* D = reinterpret_cast<char*>(dst + (r0 * 256 + c0));
        if (r0 + r < n) *reinterpret_cast<uint4*>(D + (uint32_t)(r * 512 + (lane & 3) * 16)) = q;
    };
    // Forward epilogue: bfloat16, ReLU, mask.
    auto activate = [&](int l, uint16_t (*h)[FLD]) {
        uint16_t y[2][4];
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                y[j][v] = relu_bf16(f2bf(acc[j][v]));
                mask[l] |= (bf2f(y[j][v]) > 0.0f ? 1u : 0u) << (4 * j + v);
            }
        put(h, y, io.h_out[l], io.hT[l]);
    };
    // 256-deep product of the rows in hin with the operand in wf[slot].
    auto product = [&](int slot, uint16_t (*hin)[FLD]) {
#pragma unroll
        for (int sl = 0; sl < 8; ++sl) {
            const bf16x8 a = load_bf16x8(&hin[lr][32 * sl + lk]);
#pragma unroll
            for (int j = 0; j < 2; ++j)
                acc[j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, wf[slot][j][sl], acc[j], 0, 0, 0);
        }
    };
    auto start = [&](int l) {
#pragma unroll
        for (int j = 0; j < 2; ++j)
            acc[j] = l < 0 ? f32x4{0.f, 0.f, 0.f, 0.f} : f32x4{bias[l][j], bias[l][j], bias[l][j], bias[l][j]};
    };
    // Backward epilogue: the mask of layer l, bfloat16.
    auto masked = [&](int l, uint16_t (&y)[2][4]) {
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int v = 0; v < 4; ++v) y[j][v] = f2bf((mask[l] >> (4 * j + v)) & 1u ? acc[j][v] : 0.0f);
    };

    // Layer 1.
    {
        uint16_t v[8];
        v[0] = f2bf(f0.x); v[1] = f2bf(f0.y); v[2] = f2bf(f0.z); v[3] = f2bf(f0.w);
        v[4] = f2bf(f1.x); v[5] = f2bf(f1.y); v[6] = f2bf(f1.z); v[7] = 0;
        const bf16x8 a = *reinterpret_cast<const bf16x8*>(v);
        start(0);
#pragma unroll
        for (int j = 0; j < 2; ++j) acc[j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, wf0[j], acc[j], 0, 0, 0);
        if (wave == 0 && lq == 0) {
            if (live && KEEP) *reinterpret_cast<bf16x8*>(io.x_out + (r0 + lr) * kFeatLd) = a;
            uint16_t* T = rows_of(io.xT, kFeatLd) + (lr >> 3) * kFeatLd * 8 + (lr & 7);
#pragma unroll
            for (int t = 0; t < 8; ++t) T[8 * t] = live ? v[t] : (uint16_t)0;
            if (pad)
#pragma unroll
                for (int t = 0; t < 8; ++t) T[2 * kFeatLd * 8 + 8 * t] = 0;
        }
    }
    activate(0, h1s);
    __syncthreads();
    // Layer 2; its operand's registers then take W3^T, in quarters.
    start(1);
    product(0, h1s);
    load_weights(0, io.wt[1], 0, 2);
    activate(1, h2s);
    __syncthreads();
    // Layer 3.
    load_weights(0, io.wt[1], 2, 4);
    start(2);
    product(1, h2s);
    load_weights(0, io.wt[1], 4, 6);
    activate(2, h3s);
    __syncthreads();
    load_weights(0, io.wt[1], 6, 8);
    // Layer 4, weights first: lane l (K-group 0) gets both outputs of row l
    // in elements 0 and 1.  The first operand's rows above 1 are copies that
    // feed elements nobody reads.
    f32x4 o = f32x4{b40, b41, 0.f, 0.f};
#pragma unroll
    for (int sl = 0; sl < 8; ++sl) {
        const bf16x8 a = load_bf16x8(&w4s[lr & 1][32 * sl + lk]);
        const bf16x8 b = load_bf16x8(&h3s[lr][32 * sl + lk]);
        o = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, o, 0, 0, 0);
    }
    load_weights(1, io.wt[0], 0, 2);
    // Gradient of the loss: binary cross-entropy of the logit plus Huber
    // (delta 1) of the FLI output, averaged over the n rows.
    uint16_t g40 = 0, g41 = 0;
    if (lq == 0 && live) {
        const float sig = 1.0f / (1.0f + expf(-o[0]));
        g40 = f2bf((sig - lab) / (float)n);
        g41 = f2bf(fminf(fmaxf(o[1] - tgt, -1.0f), 1.0f) / (float)n);
    }
    // g3 = (g4 W4) * (h3 > 0): K = 2, padded to one 32-deep slice.
    uint16_t y[2][4];
    {
        uint16_t v[8] = {g40, g41, 0, 0, 0, 0, 0, 0};
        const bf16x8 a = *reinterpret_cast<const bf16x8*>(v);
        start(-1);
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            uint16_t w[8] = {0, 0, 0, 0, 0, 0, 0, 0};
            if (lq == 0) { w[0] = w4s[0][c0 + 16 * j + lr]; w[1] = w4s[1][c0 + 16 * j + lr]; }
            acc[j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, *reinterpret_cast<const bf16x8*>(w), acc[j], 0, 0, 0);
        }
    }
    load_weights(1, io.wt[0], 2, 4);
    masked(2, y);
    put(g3s, y, io.g_out[2], io.gT[2]);
    __syncthreads();
    // g2 = (g3 W3) * (h2 > 0).
    load_weights(1, io.wt[0], 4, 6);
    start(-1);
    product(0, g3s);
    load_weights(1, io.wt[0], 6, 8);
    masked(1, y);
    put(h3s, y, io.g_out[1], io.gT[1]);
    __syncthreads();
    // g1 = (g2 W2) * (h1 > 0).
    start(-1);
    product(1, h3s);
    masked(0, y);
    put(h2s, y, io.g_out[0], io.gT[0]);
    // The outputs, their gradient and the loss itself, behind everything that
    // another wavefront waits for.
    if (wave == 0) {
        float l = 0.0f;
        if (lq == 0) {
            if (live) {
                const float z = o[0], f = o[1], d = f - tgt;
                l = fmaxf(z, 0.0f) - lab * z + log1pf(expf(-fabsf(z)));
                l += fabsf(d) <= 1.0f ? 0.5f * d * d : fabsf(d) - 0.5f;
                if (io.out) *reinterpret_cast<float2*>(io.out + 2 * (r0 + lr)) = make_float2(z, f);
                if (KEEP)
                    *reinterpret_cast<uint32_t*>(io.gout + 2 * (r0 + lr)) = (uint32_t)g40 | ((uint32_t)g41 << 16);
            }
            uint16_t* T = rows_of(io.g4T, 2) + (lr >> 3) * 2 * 8 + (lr & 7);
            T[0] = g40;
            T[8] = g41;
            if (pad) T[2 * 2 * 8] = T[2 * 2 * 8 + 8] = 0;
        }
#pragma unroll
        for (int off = 8; off > 0; off >>= 1) l += __shfl_xor(l, off);
        if (lane == 0) atomicAdd(io.loss, l / (float)n);
    }
}

// Inference as a two-stage pipeline over 32-row tiles, one barrier per
// tile.  Wavefronts 0-3 (the front stage) run layer 2 of tile k in step k, and
// layer 1 of tile k + 1; wavefronts 4-7 (the back stage) run layer 3 of tile k - 2
// and layer 4 of tile k - 4.  Each wavefront keeps the B fragments of ONE hidden
// layer for 64 output columns (4 column blocks x 8 K-slices; the same
// registers hold W2 in the front stage and W3 in the back), so every A
// fragment read from LDS feeds four MFMAs, and both wavefronts of a SIMD
// issue a hidden layer's MFMAs in the same step.  The hidden layer's biases
// sit in registers, layer 1's biases and the two output rows in LDS.
//
// The matrix cores set the pace only if no wavefront waits for LDS or for a
// result with nothing else to issue.  So a hidden layer is 16 groups of four
// MFMAs whose fragment was requested three groups before, the conversions and
// stores of the other blocks stand between them, and the last row block's
// epilogue is left for after the next barrier, where it covers the first
// fragments' way.  That costs a third buffer of h2 and h3 (tile modulo 3: the
// first half written in one step, the second in the next, read in the third)
// and two more steps at the end.  4,194,304 rows: 859 us with two buffers and
// unordered groups (58% of the cycles with an MFMA in flight), 799 now (68%).
// The clock under this load is lower, 2.1 GHz instead of 2.3, so fewer cycles
// shorten the time by less.
// Products, K-slice order, bias-started accumulators and the bfloat16 ReLU
// epilogue are those of k_gemm_bf16: the outputs equal the
// layer-by-layer path bit for bit.
constexpr int kInferFT = 32;

__global__ __launch_bounds__(512) void k_mlp_infer(const uint16_t* __restrict__ w0, const uint16_t* __restrict__ w1,
                                                  const uint16_t* __restrict__ w2, const uint16_t* __restrict__ w3,
                                                  const float* __restrict__ b0, const float* __restrict__ b1,
                                                  const float* __restrict__ b2, const float* __restrict__ b3,
                                                  const float* __restrict__ feat, int64_t n, float* __restrict__ out) {
    constexpr int FT = kInferFT, RB = FT / 16;
    __shared__ __attribute__((aligned(16))) uint16_t h1[2][FT][FLD];
    __shared__ __attribute__((aligned(16))) uint16_t h2[3][FT][FLD];
    __shared__ __attribute__((aligned(16))) uint16_t h3[3][FT][FLD];
    __shared__ __attribute__((aligned(16))) float bs[1][256];      // layer 1's biases
    __shared__ __attribute__((aligned(16))) uint16_t w4s[2][256];
    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
    const int lr = lane & 15, lq = lane >> 4, lk = lq * 8;
    const bool front = wave < 4;                      // uniform per wavefront
    const int c0 = 64 * (wave & 3);                   // first output column of this wavefront's layer
    if (tid < 256) bs[0][tid] = b0[tid];
    w4s[tid >> 8][tid & 255] = w3[tid];               // 512 threads, 2 x 256 weights
    // B fragments: column c0 + 16 j + lr, K values 32 s + lk .. + 8.
    const uint16_t* wl = front ? w1 : w2;
    bf16x8 wf[4][8];
#pragma unroll
    for (int j = 0; j < 4; ++j)
#pragma unroll
        for (int sl = 0; sl < 8; ++sl) wf[j][sl] = load_bf16x8(wl + (int64_t)(c0 + 16 * j + lr) * 256 + 32 * sl + lk);
    // Layer 1 fragments (front; K = 7, only the lanes of K-group 0 carry values).
    bf16x8 wf0[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        uint16_t v[8];
#pragma unroll
        for (int t = 0; t < 8; ++t)
            v[t] = (front && lq == 0 && t < 7) ? w0[(c0 + 16 * j + lr) * 7 + t] : (uint16_t)0;
        wf0[j] = *reinterpret_cast<const bf16x8*>(v);
    }
    const float bias3 = lr < 2 ? b3[lr] : 0.0f;
    // The hidden layer's biases for this lane's outputs (columns
    // c0 + 16 j + 4 lq .. + 3), the accumulators' starting values.
    f32x4 bh[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const float* bl = front ? b1 : b2;
#pragma unroll
        for (int v = 0; v < 4; ++v) bh[j][v] = bl[c0 + 16 * j + 4 * lq + v];
    }

    const int64_t ntiles = (n + FT - 1) / FT;
    const int64_t mine = blockIdx.x < ntiles ? (ntiles - 1 - (int64_t)blockIdx.x) / gridDim.x + 1 : 0;
    auto tile_of = [&](int64_t k) { return (int64_t)blockIdx.x + k * gridDim.x; };
    // Feature rows (front stage): rows past n repeat row n - 1 (never stored);
    // the lanes of K-groups 1-3 meet zero weights.
    float4 fnext[RB][2];
    auto load_feat = [&](int64_t t) {
#pragma unroll
        for (int i = 0; i < RB; ++i) {
            int64_t row = t * FT + 16 * i + lr;
            row = row < n ? row : n - 1;
            fnext[i][0] = *reinterpret_cast<const float4*>(feat + row * kFeatLd);
            fnext[i][1] = *reinterpret_cast<const float4*>(feat + row * kFeatLd + 4);
        }
    };
    // Epilogue of column block j of a 16-row block (weights as the first MFMA
    // operand: element v of lane l is tile row l % 16, column 4 (l / 16) + v of the
    // 16-column block).
    auto store = [&](uint16_t (*h)[FLD], int i, int j, const f32x4& x) {
        uint2 u;
        u.x = relu_bf16x2(pack_bf16x2(x[0], x[1]));
        u.y = relu_bf16x2(pack_bf16x2(x[2], x[3]));
        *reinterpret_cast<uint2*>(&h[16 * i + lr][c0 + 16 * j + 4 * lq]) = u;
    };
    // Row block i of the tile whose features are in fnext, as a fragment.
    auto feat_frag = [&](int i) {
        uint16_t v[8];
        v[0] = f2bf(fnext[i][0].x); v[1] = f2bf(fnext[i][0].y); v[2] = f2bf(fnext[i][0].z);
        v[3] = f2bf(fnext[i][0].w); v[4] = f2bf(fnext[i][1].x); v[5] = f2bf(fnext[i][1].y);
        v[6] = f2bf(fnext[i][1].z); v[7] = 0;
        return *reinterpret_cast<const bf16x8*>(v);
    };
    auto bias1 = [&](int j) { return *reinterpret_cast<const f32x4*>(&bs[0][c0 + 16 * j + 4 * lq]); };
    // A hidden layer of one tile (W2 in the front stage, W3 in the back) as 16
    // groups of one K slice of one row block: group m = 8 i + s takes its fragment
    // from the ring, requests that of group m + 3 and issues four MFMAs, and side(m)
    // adds the other work that belongs there.  Nothing moves between groups.
    f32x4 x[2][4];
    bf16x8 ring[4];
    auto request = [&](uint16_t (*hin)[FLD], int m) {
        ring[m & 3] = load_bf16x8(&hin[16 * (m >> 3) + lr][32 * (m & 7) + lk]);
    };
    auto hidden = [&](uint16_t (*hin)[FLD], auto&& side) {
#pragma unroll
        for (int m = 0; m < 16; ++m) {
            if (m + 3 < 16) request(hin, m + 3);
            const int i = m >> 3, sl = m & 7;
#pragma unroll
            for (int j = 0; j < 4; ++j)
                x[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wf[j][sl], ring[m & 3], sl == 0 ? bh[j] : x[i][j], 0,
                                                                  0, 0);
            side(m);
            __builtin_amdgcn_sched_barrier(0);
        }
    };
    auto begin = [&](uint16_t (*hin)[FLD]) {
        request(hin, 0);
        request(hin, 1);
        request(hin, 2);
    };
    __syncthreads();                                  // layer 1's biases and output rows in LDS
    if (front) {
        f32x4 y[4];
        auto layer1 = [&](int i) {
            const bf16x8 a = feat_frag(i);
#pragma unroll
            for (int j = 0; j < 4; ++j) y[j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wf0[j], a, y[j], 0, 0, 0);
        };
        auto bias_y = [&]() {
#pragma unroll
            for (int j = 0; j < 4; ++j) y[j] = bias1(j);
        };
        load_feat(tile_of(0));
#pragma unroll
        for (int i = 0; i < RB; ++i) {
            bias_y();
            layer1(i);
#pragma unroll
            for (int j = 0; j < 4; ++j) store(h1[0], i, j, y[j]);
        }
        load_feat(tile_of(1));
        bias_y();
        int w = 0;                                    // h2 buffer of the tile
        // Tile k: layer 2 (its second row block is stored after the next barrier),
        // and layer 1 of tile k + 1.
        auto tile = [&](auto later, int64_t k, uint16_t (*hin)[FLD], uint16_t (*h1n)[FLD], uint16_t (*hout)[FLD],
                        uint16_t (*hprev)[FLD]) {
            constexpr bool LATER = decltype(later)::value;      // a tile went before this one
            begin(hin);
            layer1(0);
            __builtin_amdgcn_sched_barrier(0);
            hidden(hin, [&](int m) {
                if (LATER && m < 4) store(hprev, 1, m, x[1][m]);
                if (m >= 2 && m < 6) store(h1n, 0, m - 2, y[m - 2]);
                if (m == 6) bias_y();
                if (m == 8) layer1(1);
                if (m == 9) load_feat(tile_of(k + 2));
                if (m >= 10 && m < 14) store(hout, 0, m - 10, x[0][m - 10]);
                if (m >= 12) store(h1n, 1, m - 12, y[m - 12]);
                if (m == 15) bias_y();
            });
        };
        __syncthreads();
        tile(std::false_type{}, 0, h1[0], h1[1], h2[0], h2[0]);
        for (int64_t k = 1; k < mine; ++k) {
            const int v = w;
            w = w == 2 ? 0 : w + 1;
            __syncthreads();
            tile(std::true_type{}, k, h1[k & 1], h1[1 - (k & 1)], h2[w], h2[v]);
        }
        __syncthreads();
#pragma unroll
        for (int j = 0; j < 4; ++j) store(h2[w], 1, j, x[1][j]);
        __syncthreads();
        __syncthreads();
        __syncthreads();
    } else {
        // Layer 4, row block wave - 4: outputs 0 and 1 in columns 0 and 1; the other
        // lanes' B operands (copies of row lane % 2) feed columns that are never
        // stored.
        auto back = [&](auto last) {
            constexpr bool LAST = decltype(last)::value;       // this wavefront runs layer 4
            const int i4 = LAST ? wave - 4 : 0;
            f32x4 o;
            // The operands of slice s are requested two groups before their MFMA.
            bf16x8 a4[2], w4[2];
            auto request4 = [&](uint16_t (*h)[FLD], int sl) {
                a4[sl & 1] = load_bf16x8(&h[16 * i4 + lr][32 * sl + lk]);
                w4[sl & 1] = load_bf16x8(&w4s[lr & 1][32 * sl + lk]);
            };
            auto layer4 = [&](int sl) {
                o = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
                    a4[sl & 1], w4[sl & 1], sl == 0 ? f32x4{bias3, bias3, bias3, bias3} : o, 0, 0, 0);
            };
            auto output = [&](int64_t t) {
                if (lr < 2) {
#pragma unroll
                    for (int v = 0; v < 4; ++v) {
                        const int64_t row = t * FT + 16 * i4 + 4 * lq + v;
                        if (row < n) out[row * 2 + lr] = o[v];
                    }
                }
            };
            auto tile = [&](auto later, uint16_t (*hin)[FLD], uint16_t (*hout)[FLD], uint16_t (*hprev)[FLD],
                            uint16_t (*h4)[FLD]) {
                constexpr bool LATER = decltype(later)::value;
                begin(hin);
                hidden(hin, [&](int m) {
                    if (LATER && m < 4) store(hprev, 1, m, x[1][m]);
                    if (LATER && LAST) {              // slice s: requested in group s, used in s + 2
                        if (m >= 2 && m < 10) layer4(m - 2);
                        if (m < 8) request4(h4, m);
                    }
                    if (m >= 10 && m < 14) store(hout, 0, m - 10, x[0][m - 10]);
                });
            };
            int w = 0;                                // h2 and h3 buffer of the tile
            __syncthreads();
            __syncthreads();
            __syncthreads();
            tile(std::false_type{}, h2[0], h3[0], h3[0], h3[0]);
            for (int64_t t = 1; t < mine; ++t) {
                const int v = w, l4 = w == 0 ? 2 : w - 1;      // tiles t - 1 and t - 2
                w = w == 2 ? 0 : w + 1;
                __syncthreads();
                tile(std::true_type{}, h2[w], h3[w], h3[v], h3[l4]);
                if (LAST && t >= 2) output(tile_of(t - 2));
            }
            __syncthreads();
#pragma unroll
            for (int j = 0; j < 4; ++j) store(h3[w], 1, j, x[1][j]);
            if (LAST && mine >= 2) {
#pragma unroll
                for (int sl = 0; sl < 8; ++sl) { request4(h3[w == 0 ? 2 : w - 1], sl); layer4(sl); }
                output(tile_of(mine - 2));
            }
            __syncthreads();
            if (LAST) {
#pragma unroll
                for (int sl = 0; sl < 8; ++sl) { request4(h3[w], sl); layer4(sl); }
                output(tile_of(mine - 1));
            }
        };
        if (wave - 4 < RB) back(std::true_type{});
        else back(std::false_type{});
    }
}

// The second half of a training step: weight gradients dW_l = g_l^T a_(l-1)
// and bias gradients (column sums of g_l) over the batch rows, and the Adam
// update of the elements they belong to, with the bfloat16 copies.
struct UpdateArgs {
    Blocks g[4];            // g1 .. g4 (256, 256, 256, 2 columns)
    Blocks a[4];            // X, h1, h2, h3 (8, 256, 256, 256 columns)
    int full, slices;       // whole slices, and all
    int chunk[4];           // 32-row slices of a split of layer l's sums
    int splits[4];
    float *w[4], *mw[4], *vw[4];
    float *b[4], *mb[4], *vb[4];
    uint16_t* wb[4];
    uint16_t* w0p;          // W1 [256][8]
    uint16_t* wf[2];        // W2, W3 in fragment order
    uint16_t* wt[2];        // W2, W3 transposed in fragment order
    float lr, c1, c2;       // c1 = 1 - b1^t, c2 = 1 - b2^t
};

// Adam on one element; returns the new weight.
__device__ __forceinline__ float adam(float g, float* w, float* pm, float* pv, int64_t e, float lr, float c1,
                                      float c2) {
    const float m = 0.9f * pm[e] + 0.1f * g;
    const float v = 0.999f * pv[e] + 0.001f * g * g;
    pm[e] = m;
    pv[e] = v;
    const float x = w[e] - lr * (m / c1) / (sqrtf(v / c2) + 1e-8f);
    w[e] = x;
    return x;
}

// Sums over the 32-row slices [s0, s1) of the products of MB x NB blocks of 16
// columns: acc[i][j] += sum G(row, m0 + 16 i + .) A(row, n0 + 16 j + .), slices in
// increasing order, one 16x16x32 MFMA each.  Operands in row-block order are
// in fragment order as they lie: lane l takes the eight rows 32 s + 8 (l / 16) ..
// of its column, 16 bytes, and 16 lanes read 256 bytes in a row.  Columns from
// cg (ca) on are zero.
template <int MB, int NB>
__device__ __forceinline__ void slice_sums(const uint16_t* G, int cg, int m0, const uint16_t* A, int ca, int n0,
                                           int s0, int s1, int lane, f32x4 (&acc)[MB][NB]) {
    const int lr = lane & 15, lq = lane >> 4;
    const bf16x8 zero = {};
    for (int s = s0; s < s1; s += 4) {
        bf16x8 x[4][MB], y[4][NB];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const bool in = s + q < s1;
            const int64_t rb = (int64_t)(s + q) * 4 + lq;
#pragma unroll
            for (int i = 0; i < MB; ++i) {
                const int c = m0 + 16 * i + lr;
                x[q][i] = in && c < cg ? load_bf16x8(G + (rb * cg + c) * 8) : zero;
            }
#pragma unroll
            for (int j = 0; j < NB; ++j) {
                const int c = n0 + 16 * j + lr;
                y[q][j] = in && c < ca ? load_bf16x8(A + (rb * ca + c) * 8) : zero;
            }
        }
#pragma unroll
        for (int q = 0; q < 4; ++q)
            if (s + q < s1) {
#pragma unroll
                for (int i = 0; i < MB; ++i)
#pragma unroll
                    for (int j = 0; j < NB; ++j)
                        acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(x[q][i], y[q][j], acc[i][j], 0, 0, 0);
            }
    }
}

constexpr int kUpWaves = 16;        // wavefronts of an update workgroup
constexpr int kPartLd = 36;         // row stride of a partial tile in LDS: lanes of all four K-groups on their own banks
constexpr int kHiddenTiles = 64;    // 32 x 32 tiles of a hidden weight

// Layer l's gradient of the 16 MB x 16 NB tile at (m0, n0): wavefront w sums
// split w (and w + 16, ..), the partials meet in LDS, and thread t returns
// element (t / 32, t % 32) summed over the splits in increasing order.
template <int MB, int NB, bool APART>
__device__ __forceinline__ float tile_gradient(const UpdateArgs& u, int l, int cg, int m0, int ca, int n0,
                                               float (*part)[32 * kPartLd]) {
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
    const int lr = lane & 15, lq = lane >> 4;
    const int slices = u.slices, chunk = u.chunk[l], splits = u.splits[l];
    const int r = tid >> 5, c = tid & 31;
    float x = 0.0f;
    for (int z0 = 0; z0 < splits; z0 += kUpWaves) {
        const int z = z0 + wave;
        if (z < splits) {
            f32x4 acc[MB][NB];
#pragma unroll
            for (int i = 0; i < MB; ++i)
#pragma unroll
                for (int j = 0; j < NB; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
            const int s1 = (z + 1) * chunk < slices ? (z + 1) * chunk : slices;
            slice_sums<MB, NB>(u.g[l].full, cg, m0, u.a[l].full, ca, n0, z * chunk, APART && s1 > u.full ? u.full : s1,
                               lane, acc);
            if (APART && s1 > u.full) slice_sums<MB, NB>(u.g[l].last, cg, m0, u.a[l].last, ca, n0, 0, 1, lane, acc);
#pragma unroll
            for (int i = 0; i < MB; ++i)
#pragma unroll
                for (int j = 0; j < NB; ++j)
#pragma unroll
                    for (int v = 0; v < 4; ++v)
                        part[wave][(16 * i + 4 * lq + v) * kPartLd + 16 * j + lr] = acc[i][j][v];
        }
        __syncthreads();
        if (r < 16 * MB && c < 16 * NB) {
            const int left = splits - z0;
#pragma unroll
            for (int q = 0; q < kUpWaves; ++q)
                if (q < left) x += part[q][r * kPartLd + c];
        }
        if (z0 + kUpWaves < splits) __syncthreads();
    }
    return x;
}

// Workgroups: kHiddenTiles per hidden weight (32 x 32 tiles), 8 for W1 (32
// rows each), 8 for W4 (32 columns each), then the biases, 32 columns each (8 per
// hidden layer, one for the output layer).  A tile is complete in its
// workgroup, so its Adam update follows at once: no partial sums in memory and
// no second launch (before: 15.7 us for the products with split partials of 8 MB,
// 8.5 us for Adam, at 2,048 rows; 6.8 us together now).  Bound by the operands'
// way from the other XCDs' L2 and by latency: 16 wavefronts keep 16 KB each in
// flight.  Consecutive workgroups go to different XCDs, so workgroup b takes its
// tile from the 4 x 4 block of tiles of XCD b % 8, which reads 1 MB of
// operands instead of 2.
constexpr int kUpW1 = 2 * kHiddenTiles, kUpW4 = kUpW1 + 8, kUpBias = kUpW4 + 8, kUpBlocks = kUpBias + 25;

// APART: the last slice, not whole, is apart from the others (a choice of address
// per slice instead took 20% more at 8,200 rows: fewer loads in flight).
template <bool APART>
__global__ __launch_bounds__(1024) void k_mlp_update(UpdateArgs u) {
    __shared__ __attribute__((aligned(16))) float part[kUpWaves][32 * kPartLd];
    __shared__ __attribute__((aligned(16))) uint16_t tile[32][40];
    const int tid = threadIdx.x, b = blockIdx.x;
    const int r = tid >> 5, c = tid & 31;
    if (b < kUpW1) {
        const int x = b & 7, q = b >> 3;                 // XCD, tile of its 4 x 4 block
        const int l = 1 + (x >> 2);
        const int m0 = 32 * (4 * (x & 1) + (q & 3)), n0 = 32 * (4 * ((x >> 1) & 1) + (q >> 2));
        const float g = tile_gradient<2, 2, APART>(u, l, 256, m0, 256, n0, part);
        const int64_t e = (int64_t)(m0 + r) * 256 + n0 + c;
        const uint16_t y = f2bf(adam(g, u.w[l], u.mw[l], u.vw[l], e, u.lr, u.c1, u.c2));
        u.wb[l][e] = y;
        tile[r][c] = y;
        __syncthreads();
        // The tile is two fragments of W (32 columns m, one K slice n) and two of
        // W^T (32 columns n, one K slice m): one 16-byte piece per thread.
        if (tid < 256) {
            const int f = (tid >> 6) & 1, lane = tid & 63, lr = lane & 15, lk = (lane >> 4) * 8;
            union { uint4 v; uint16_t e[8]; } p;
#pragma unroll
            for (int t = 0; t < 8; ++t) p.e[t] = tid < 128 ? tile[16 * f + lr][lk + t] : tile[lk + t][16 * f + lr];
            uint16_t* F = tid < 128 ? u.wf[l - 1] + (((m0 / 16 + f) * 8 + n0 / 32) * 64 + lane) * 8
                                    : u.wt[l - 1] + (((n0 / 16 + f) * 8 + m0 / 32) * 64 + lane) * 8;
            *reinterpret_cast<uint4*>(F) = p.v;
        }
        return;
    }
    if (b < kUpBias) {
        const bool first = b < kUpW4;
        const int k = 32 * (first ? b - kUpW1 : b - kUpW4), l = first ? 0 : 3;
        const float g = first ? tile_gradient<2, 1, APART>(u, 0, 256, k, kFeatLd, 0, part)
                              : tile_gradient<1, 2, APART>(u, 3, 2, 0, 256, k, part);
        if (first ? c < 7 : r < 2) {
            const int64_t e = first ? (int64_t)(k + r) * 7 + c : (int64_t)r * 256 + k + c;
            const uint16_t y = f2bf(adam(g, u.w[l], u.mw[l], u.vw[l], e, u.lr, u.c1, u.c2));
            u.wb[l][e] = y;
            if (first) u.w0p[(k + r) * 8 + c] = y;
        }
        return;
    }
    // Bias columns: thread (r, c) sums rows 8 r + t + 256 q of column c over q, one
    // sum per t < 8, and the 256 sums of a column meet pairwise, halves first.
    const int l = (b - kUpBias) >> 3, n0 = 32 * ((b - kUpBias) & 7), cols = kOut[l];
    float s[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    if (n0 + c < cols) {
        auto add = [&](const uint16_t* G, int64_t rb) {
            union { bf16x8 v; uint16_t e[8]; } p;
            p.v = load_bf16x8(G + (rb * cols + n0 + c) * 8);
#pragma unroll
            for (int t = 0; t < 8; ++t) s[t] += bf2f(p.e[t]);
        };
        const int end = 4 * (APART ? u.full : u.slices);
        int rb = r;
        for (; rb < end; rb += 32) add(u.g[l].full, rb);
        if (APART && rb < end + 4) add(u.g[l].last, rb - end);
    }
    float (*half)[32][8] = reinterpret_cast<float (*)[32][8]>(&part[0][0]);
    for (int k = 16; k > 0; k >>= 1) {
        if (r >= k && r < 2 * k)
#pragma unroll
            for (int t = 0; t < 8; ++t) half[r - k][c][t] = s[t];
        __syncthreads();
        if (r < k)
#pragma unroll
            for (int t = 0; t < 8; ++t) s[t] += half[r][c][t];
        __syncthreads();
    }
    if (r == 0 && n0 + c < cols) {
#pragma unroll
        for (int k = 4; k > 0; k >>= 1)
#pragma unroll
            for (int t = 0; t < k; ++t) s[t] += s[t + k];
        adam(s[0], u.b[l], u.mb[l], u.vb[l], n0 + c, u.lr, u.c1, u.c2);
    }
}

// The tensors of a step in row-major order, dst, from their row-block order, whose
// whole slices lie in dst itself: eight rows take the same bytes in both orders, so
// a workgroup reads 2,048 elements of whole 8-row blocks, exchanges them in LDS and
// writes them to the same place (those of the slice at `last`: to its rows in dst).
// Grid (8-row blocks of 256 columns, tensors); 8,192 rows: 25 MB each way.
struct RowMajorArgs {
    Blocks t[8];
    uint16_t* dst[8];
    int cols[8];            // powers of two, at most 256
    int64_t n;
};

__global__ __launch_bounds__(256) void k_row_major(RowMajorArgs p) {
    __shared__ __attribute__((aligned(16))) uint16_t tile[2048];
    const int k = blockIdx.y, tid = threadIdx.x, C = p.cols[k];
    const int64_t total = p.n * C, base = (int64_t)blockIdx.x * 2048;
    if (base >= total) return;                        // the same in all threads
    const int64_t full = (p.n >> 5) * 32 * C;         // elements of the whole slices
    const int64_t e = base + 8 * tid;                 // this thread's column of an 8-row block
    if (e < (p.n + 7) / 8 * 8 * C) {
        union { uint4 v; uint16_t e[8]; } u;
        u.v = *reinterpret_cast<const uint4*>(e < full ? p.t[k].full + e : p.t[k].last + (e - full));
        const int g = tid / C, c = tid % C;
#pragma unroll
        for (int r = 0; r < 8; ++r) tile[(8 * g + r) * C + c] = u.e[r];
    }
    __syncthreads();
    if (e + 8 <= total)
        *reinterpret_cast<uint4*>(p.dst[k] + e) = *reinterpret_cast<const uint4*>(&tile[8 * tid]);
    else
        for (int r = 0; r < 8 && e + r < total; ++r) p.dst[k][e + r] = tile[8 * tid + r];
}

// The training pass's copies of the weights (grid 520 x 256 threads: one
// element of W2, W3 or the padded W1 each), formed once before a run of steps;
// the updates keep them.
__global__ __launch_bounds__(256) void k_pack_weights(const uint16_t* w0, const uint16_t* w1, const uint16_t* w2,
                                                      uint16_t* w0p, uint16_t* f1, uint16_t* f2, uint16_t* t1,
                                                      uint16_t* t2) {
    const int e = blockIdx.x * 256 + threadIdx.x;
    if (e >= 131072) {
        const int o = (e - 131072) >> 3, i = e & 7;
        w0p[e - 131072] = i < 7 ? w0[o * 7 + i] : (uint16_t)0;
        return;
    }
    const int o = (e >> 8) & 255, i = e & 255;
    const uint16_t x = (e < 65536 ? w1 : w2)[e & 65535];
    auto at = [](int col, int k) { return (((col >> 4) * 8 + (k >> 5)) * 64 + ((k >> 3) & 3) * 16 + (col & 15)) * 8 + (k & 7); };
    (e < 65536 ? f1 : f2)[at(o, i)] = x;
    (e < 65536 ? t1 : t2)[at(i, o)] = x;
}

__global__ __launch_bounds__(256) void k_to_bf16(const float* x, int64_t n, uint16_t* y) {
    const int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (e < n) y[e] = f2bf(x[e]);
}

// Standardised features of scan points: (beta, chi1, chi2, r0, cos th1,
// cos th2, log10 t_end), each (x - mean) / std; column 7 is zero padding.
struct FeatArgs {
    const double *beta, *chi1, *chi2;
    double beta0, chi1_0, chi2_0;
    const double *r0, *th1, *th2, *t_end;
    double t_end_all;
    const int32_t* idx;     // rows to take (null: all)
    int64_t n;
    float mean[7], stdv[7];
    float* feat;
};

__global__ __launch_bounds__(256) void k_features(FeatArgs f) {
    const int64_t j = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (j >= f.n) return;
    const int64_t i = f.idx ? (int64_t)f.idx[j] : j;
    double x[7];
    x[0] = f.beta ? f.beta[i] : f.beta0;
    x[1] = f.chi1 ? f.chi1[i] : f.chi1_0;
    x[2] = f.chi2 ? f.chi2[i] : f.chi2_0;
    x[3] = f.r0[i];
    x[4] = cos(f.th1[i]);
    x[5] = cos(f.th2[i]);
    x[6] = log10(f.t_end ? f.t_end[i] : f.t_end_all);
#pragma unroll
    for (int c = 0; c < 7; ++c) f.feat[j * kFeatLd + c] = (float)((x[c] - f.mean[c]) / f.stdv[c]);
    f.feat[j * kFeatLd + 7] = 0.0f;
}

// Training targets from a scan: label 1.0 chaotic / 0.0 otherwise, and the
// FLI relative to log10 t_end (0 for orbits whose FLI is not finite).
__global__ __launch_bounds__(256) void k_targets(const double* fli, const int8_t* label, const double* t_end,
                                                 double t_end_all, int64_t n, float* lab, float* target) {
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= n) return;
    lab[i] = label[i] == 1 ? 1.0f : 0.0f;
    const double t = t_end ? t_end[i] : t_end_all;
    const double f = fli[i];
    target[i] = isfinite(f) ? (float)(f - log10(t)) : 0.0f;
}

// SplitMix64 (Steele, Lea & Flood 2014): the audit draw of point i.
__device__ __forceinline__ uint64_t splitmix64(uint64_t x) {
    x += 0x9e3779b97f4a7c15ull;
    x = (x ^ (x >> 30)) * 0xbf58476d1ce4e5b9ull;
    x = (x ^ (x >> 27)) * 0x94d049bb133111ebull;
    return x ^ (x >> 31);
}

__global__ void k_clear_count(unsigned long long* c) { c[threadIdx.x] = 0ull; }

// Surrogate label sign(logit); points with |logit| < margin or drawn for the
// audit (SplitMix64(seed + i) / 2^64 < audit) join the integration list.
__global__ __launch_bounds__(256) void k_gate(const float* out, int64_t n, float margin, double audit,
                                              unsigned long long seed, int8_t* label, float* fli_pred,
                                              int32_t* list, unsigned long long* count) {
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= n) return;
    const float z = out[2 * i];
    label[i] = z > 0.0f ? 1 : 0;
    if (fli_pred) fli_pred[i] = out[2 * i + 1];
    const double u = (double)(splitmix64(seed + (uint64_t)i) >> 11) * 0x1.0p-53;
    if (fabsf(z) < margin || u < audit) {
        const unsigned long long pos = atomicAdd(count, 1ull);
        list[pos] = (int32_t)i;
    }
}

__device__ __forceinline__ bool audit_draw(uint64_t seed, int64_t i, double audit) {
    return (double)(splitmix64(seed + (uint64_t)i) >> 11) * 0x1.0p-53 < audit;
}

// The audit sample alone: points with SplitMix64(seed + i) / 2^64 < audit,
// listed by increasing index: points per workgroup, the places where the
// workgroups' points begin, and the list itself.  Appending with an atomic per
// point took 50 us for 5,000 of 524,288 points, and the list then had to be
// sorted on the host, with two copies; with these three the whole assisted scan
// of those points takes 10.75 ms instead of 10.98.
constexpr int kAuditItems = 8, kAuditPoints = 256 * kAuditItems;    // per lane, per workgroup

// Bit q: point i0 + q is drawn.
__device__ __forceinline__ uint32_t audit_bits(uint64_t seed, int64_t i0, int64_t n, double audit) {
    uint32_t bits = 0;
#pragma unroll
    for (int q = 0; q < kAuditItems; ++q)
        if (i0 + q < n && audit_draw(seed, i0 + q, audit)) bits |= 1u << q;
    return bits;
}

// Sum of v over the lanes of the workgroup before this one; total: over all.
template <int THREADS>
__device__ __forceinline__ uint32_t block_prefix(uint32_t v, uint32_t* part, uint32_t& total) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    uint32_t x = v;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        const uint32_t y = __shfl_up(x, off);
        if (lane >= off) x += y;
    }
    __syncthreads();                        // part may still be read from an earlier call
    if (lane == 63) part[wave] = x;
    __syncthreads();
    uint32_t before = 0, all = 0;
#pragma unroll
    for (int w = 0; w < THREADS / 64; ++w) {
        if (w < wave) before += part[w];
        all += part[w];
    }
    total = all;
    return before + x - v;
}

__global__ __launch_bounds__(256) void k_audit_count(int64_t n, double audit, unsigned long long seed,
                                                     uint32_t* first) {
    __shared__ uint32_t part[4];
    const int64_t i0 = (int64_t)blockIdx.x * kAuditPoints + threadIdx.x * kAuditItems;
    uint32_t total;
    block_prefix<256>(__popc(audit_bits(seed, i0, n, audit)), part, total);
    if (threadIdx.x == 0) first[blockIdx.x] = total;
}

// first[b]: points of workgroup b -> points before it; count: all.
__global__ __launch_bounds__(1024) void k_audit_scan(uint32_t* first, int64_t blocks, unsigned long long* count) {
    __shared__ uint32_t part[16];
    uint32_t base = 0;
    for (int64_t b0 = 0; b0 < blocks; b0 += 1024) {
        const int64_t b = b0 + threadIdx.x;
        uint32_t total;
        const uint32_t before = block_prefix<1024>(b < blocks ? first[b] : 0u, part, total);
        if (b < blocks) first[b] = base + before;
        base += total;
    }
    if (threadIdx.x == 0) *count = base;
}

__global__ __launch_bounds__(256) void k_audit_list(int64_t n, double audit, unsigned long long seed,
                                                    const uint32_t* first, int32_t* list) {
    __shared__ uint32_t part[4];
    const int64_t i0 = (int64_t)blockIdx.x * kAuditPoints + threadIdx.x * kAuditItems;
    const uint32_t bits = audit_bits(seed, i0, n, audit);
    uint32_t total;
    uint32_t at = first[blockIdx.x] + block_prefix<256>(__popc(bits), part, total);
#pragma unroll
    for (int q = 0; q < kAuditItems; ++q)
        if ((bits >> q) & 1u) list[at++] = (int32_t)(i0 + q);
}

// Network labels, and the uncertain points (|logit| < margin) that the audit
// has not already drawn.
__global__ __launch_bounds__(256) void k_gate_uncertain(const float* out, int64_t n, float margin, double audit,
                                                        unsigned long long seed, int8_t* label, int32_t* list,
                                                        unsigned long long* count) {
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= n) return;
    const float z = out[2 * i];
    label[i] = z > 0.0f ? 1 : 0;
    if (fabsf(z) < margin && !audit_draw(seed, i, audit)) list[atomicAdd(count, 1ull)] = (int32_t)i;
}

// dst[j] = src[idx[j]] (src NULL: fill).
__global__ __launch_bounds__(256) void k_gather_f64(const double* src, double fill, const int32_t* idx, int64_t m,
                                                    double* dst) {
    const int64_t j = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (j < m) dst[j] = src ? src[idx[j]] : fill;
}

__global__ __launch_bounds__(256) void k_merge(const int32_t* list, int64_t m, const int8_t* integrated,
                                               int8_t* label) {
    const int64_t j = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (j < m) label[list[j]] = integrated[j];
}

// *total += steps[0] + ... + steps[m - 1]: a grid-stride partial sum per
// lane, a workgroup sum in LDS, one atomic per workgroup.
__global__ __launch_bounds__(256) void k_sum_steps(const int64_t* steps, int64_t m, unsigned long long* total) {
    __shared__ unsigned long long part[256];
    unsigned long long s = 0;
    for (int64_t j = (int64_t)blockIdx.x * 256 + threadIdx.x; j < m; j += (int64_t)gridDim.x * 256)
        s += (unsigned long long)steps[j];
    part[threadIdx.x] = s;
    __syncthreads();
    for (int w = 128; w > 0; w >>= 1) {
        if ((int)threadIdx.x < w) part[threadIdx.x] += part[threadIdx.x + w];
        __syncthreads();
    }
    if (threadIdx.x == 0) atomicAdd(total, part[0]);
}

unsigned blocks_for(int64_t n, int per) { return (unsigned)((n + per - 1) / per); }

void gemm(hipStream_t s, int M, int N, int K, const uint16_t* A, int64_t sam, int64_t sak, const uint16_t* B,
          int64_t sbk, int64_t sbn, const float* bias, int relu, const uint16_t* mask, int64_t ldm, float* Cf,
          int64_t ldcf, uint16_t* Cb, int64_t ldcb) {
    GemmArgs g;
    g.M = M; g.N = N; g.K = K;
    g.A = A; g.sam = sam; g.sak = sak;
    g.B = B; g.sbk = sbk; g.sbn = sbn;
    g.bias = bias; g.relu = relu; g.mask = mask; g.ldm = ldm;
    g.Cf = Cf; g.ldcf = ldcf; g.Cb = Cb; g.ldcb = ldcb;
    g.amode = stage_mode(A, sam, sak);
    g.bmode = stage_mode(B, sbn, sbk);
    hipLaunchKernelGGL(k_gemm_bf16, dim3(blocks_for(N, BN), blocks_for(M, BM)), dim3(256), 0, s, g);
}

pn_status launched(const char* what) {
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) {
        pn_detail::set_last_error(what, hipGetErrorString(e));
        return PN_EDEVICE;
    }
    return PN_OK;
}

size_t al(size_t x) { return (x + 255) & ~(size_t)255; }

size_t rows32(int batch) { return ((size_t)batch + 31) / 32 * 32; }

// Bytes of a training workspace behind the reported tensors, the same for every
// batch (callers keep workspaces of this size).
constexpr size_t kStepRoom = 17576960;

// Whether the row-block tensors of a step have room behind the reported ones (up
// to 5,504 rows).  Otherwise they take those tensors' places.
bool blocks_apart(int batch) {
    const size_t R = rows32(batch);
    return al(R * kFeatLd * 2) + 6 * al(R * 256 * 2) + al(R * 2 * 2) + 4 * al(256 * 256 * 2) + al(256 * 8 * 2) <= kStepRoom;
}

bool net_ok(const pn_mlp* net, bool training) {
    if (!net) return false;
    for (int l = 0; l < 4; ++l) {
        if (!net->w[l] || !net->b[l] || !net->wb[l]) return false;
        if (training && (!net->mw[l] || !net->vw[l] || !net->mb[l] || !net->vb[l])) return false;
    }
    return true;
}

// Inference over n rows (persistent grid of at most one workgroup per CU).
void launch_infer(hipStream_t s, const pn_mlp* net, const float* feat, int64_t n, float* out, int ncu) {
    if (n <= 0) return;
    const int64_t ntiles = (n + kInferFT - 1) / kInferFT;
    const unsigned grid = (unsigned)(ntiles < ncu ? ntiles : ncu);
    hipLaunchKernelGGL(k_mlp_infer, dim3(grid), dim3(512), 0, s, net->wb[0], net->wb[1], net->wb[2], net->wb[3],
                       net->b[0], net->b[1], net->b[2], net->b[3], feat, n, out);
}

int device_cu_count() {
    int dev = 0, ncu = 0;
    if (hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&ncu, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess)
        return 0;
    return ncu;
}

// Forward pass of rows [0, rows) whose bfloat16 inputs are in X (ld 8).
void forward(hipStream_t s, const pn_mlp* net, int64_t rows, const uint16_t* X, uint16_t* h1, uint16_t* h2,
             uint16_t* h3, float* out) {
    const int M = (int)rows;
    gemm(s, M, 256, 7, X, kFeatLd, 1, net->wb[0], 1, 7, net->b[0], 1, nullptr, 0, nullptr, 0, h1, 256);
    gemm(s, M, 256, 256, h1, 256, 1, net->wb[1], 1, 256, net->b[1], 1, nullptr, 0, nullptr, 0, h2, 256);
    gemm(s, M, 256, 256, h2, 256, 1, net->wb[2], 1, 256, net->b[2], 1, nullptr, 0, nullptr, 0, h3, 256);
    gemm(s, M, 2, 256, h3, 256, 1, net->wb[3], 1, 256, net->b[3], 0, nullptr, 0, out, 2, nullptr, 0);
}

}  // namespace

extern "C" {

size_t pn_mlp_param_count(int32_t layer, int32_t which) {
    if (layer < 0 || layer > 3) return 0;
    return which == 0 ? (size_t)kIn[layer] * kOut[layer] : (size_t)kOut[layer];
}

size_t pn_mlp_train_workspace_size(int32_t batch) {
    if (batch <= 0) return 0;
    const size_t B = (size_t)batch;
    return al(B * kFeatLd * 2) + 3 * al(B * 256 * 2) + al(B * 2 * 4) + al(B * 2 * 2) + 3 * al(B * 256 * 2) + kStepRoom;
}

pn_status pn_mlp_train_workspace_layout(int32_t batch, size_t* off) {
    if (batch <= 0 || !off) return PN_EINVAL;
    const size_t B = (size_t)batch;
    const size_t sizes[9] = {B * kFeatLd * 2, B * 256 * 2, B * 256 * 2, B * 256 * 2, B * 2 * 4, B * 2 * 2,
                             B * 256 * 2, B * 256 * 2, B * 256 * 2};
    size_t at = 0;
    for (int k = 0; k < 9; ++k) {
        off[k] = at;
        at += al(sizes[k]);
    }
    return PN_OK;
}

pn_status pn_mlp_sync_bf16(pn_mlp* net, hipStream_t stream) {
    if (!net_ok(net, false)) return PN_EINVAL;
    for (int l = 0; l < 4; ++l) {
        const int64_t n = (int64_t)kIn[l] * kOut[l];
        hipLaunchKernelGGL(k_to_bf16, dim3(blocks_for(n, 256)), dim3(256), 0, stream, net->w[l], n, net->wb[l]);
    }
    return launched("pn_mlp_sync_bf16");
}

}  // extern "C"

namespace {

// Splits of layer l's weight-gradient sums over the batch rows (32-row
// slices per split, splits): from 512 rows on as many as leave each at least 128
// rows, up to 16 for a hidden weight, one per wavefront of an update workgroup,
// and 64 for the outer two, which have fewer workgroups to share the rows.  The
// sums are formed split by split in increasing order, so this rule is part of
// the result.
void gradient_splits(int l, int batch, int& chunk, int& splits) {
    const int64_t K = batch, most = l == 1 || l == 2 ? 16 : 64;
    const int64_t sp = K >= 512 ? std::min(most, K / 128) : 1;
    chunk = (int)(((K + sp - 1) / sp + 31) / 32);
    splits = (int)((K + 32 * (int64_t)chunk - 1) / (32 * (int64_t)chunk));
}

// One training step (pn_mlp_train_step).  The workspace also holds the step's
// tensors in row-block order and bfloat16 copies of W2 and W3, straight and
// transposed, in fragment order; each update rewrites the copies with the
// bfloat16 weights, so a run of steps on one workspace forms them once (fresh)
// before its first step.  keep: the caller can read the step's tensors.  Where the
// row-block tensors lie in the places of the row-major ones (blocks_apart), these
// are formed from them at the end.  That costs a launch, in a step whose tensors
// are kept only, and saves the second place: a single step of 8,192 rows 51.5 ->
// 61.8 us and a workspace of 51.3 -> 43.0 MB, of 65,536 rows 295 -> 299 us and 406 ->
// 221 MB; 16 steps of one call 649 -> 653 and 3,734 -> 3,712 us.
pn_status train_step(pn_mlp* net, const float* feat, const float* label, const float* target, const int32_t* idx,
                     int32_t batch, int32_t step, float lr, float* loss, void* ws, size_t ws_bytes,
                     hipStream_t stream, bool fresh, bool keep) {
    if (!net_ok(net, true) || !feat || !label || !target || !idx || !loss) return PN_EINVAL;
    if ((reinterpret_cast<uintptr_t>(feat) & 15u) != 0) return PN_EINVAL;
    if (batch <= 0 || step < 1 || !(lr > 0.0f) || !std::isfinite(lr)) return PN_EINVAL;
    if (!ws || ws_bytes < pn_mlp_train_workspace_size(batch)) return PN_ENOWS;
    const int ncu = device_cu_count();
    if (ncu <= 0) {
        pn_detail::set_last_error("pn_mlp_train_step", "no device");
        return PN_EDEVICE;
    }
    const int B = batch;
    // The tensors a step leaves in the workspace, at the offsets that
    // pn_mlp_train_workspace_layout reports; the other copies follow.
    size_t off[9];
    if (pn_mlp_train_workspace_layout(batch, off) != PN_OK) return PN_EINVAL;
    char* const w0 = static_cast<char*>(ws);
    char* p = w0 + off[8] + al((size_t)B * 256 * 2);
    auto take = [&](size_t elements) { uint16_t* q = (uint16_t*)p; p += al(2 * elements); return q; };
    const bool apart = blocks_apart(B);
    const int full = B / 32;
    const size_t R = rows32(B);
    // Tensor at offset o of the workspace with C columns, in row-block order.
    auto blocks = [&](size_t o, int C) {
        if (!apart) return Blocks{(uint16_t*)(w0 + o), take(32 * (size_t)C)};
        uint16_t* const t = take(R * C);
        return Blocks{t, t + (size_t)full * 32 * C};
    };
    TrainIO io;
    UpdateArgs u;
    io.w3 = net->wb[3];
    io.feat = feat; io.label = label; io.target = target; io.idx = idx;
    io.n = B;
    io.out = keep ? (float*)(w0 + off[4]) : nullptr;
    io.loss = loss;
    io.x_out = (uint16_t*)(w0 + off[0]);
    io.gout = (uint16_t*)(w0 + off[5]);
    u.a[0] = io.xT = blocks(off[0], kFeatLd);
    u.g[3] = io.g4T = blocks(off[5], 2);
    for (int l = 0; l < 3; ++l) {
        io.h_out[l] = (uint16_t*)(w0 + off[1 + l]);
        io.g_out[l] = (uint16_t*)(w0 + off[8 - l]);
        u.a[l + 1] = io.hT[l] = blocks(off[1 + l], 256);
        u.g[l] = io.gT[l] = blocks(off[8 - l], 256);
    }
    for (int t = 0; t < 2; ++t) {
        io.wf[t] = u.wf[t] = take(256 * 256);
        io.wt[t] = u.wt[t] = take(256 * 256);
    }
    io.w0 = u.w0p = take(256 * 8);
    u.full = full;
    u.slices = (int)(R / 32);
    for (int l = 0; l < 4; ++l) {
        io.b[l] = net->b[l];
        gradient_splits(l, B, u.chunk[l], u.splits[l]);
        u.w[l] = net->w[l]; u.mw[l] = net->mw[l]; u.vw[l] = net->vw[l]; u.wb[l] = net->wb[l];
        u.b[l] = net->b[l]; u.mb[l] = net->mb[l]; u.vb[l] = net->vb[l];
    }
    u.lr = lr;
    u.c1 = 1.0f - powf(0.9f, (float)step);
    u.c2 = 1.0f - powf(0.999f, (float)step);
    if (fresh)
        hipLaunchKernelGGL(k_pack_weights, dim3(520), dim3(256), 0, stream, net->wb[0], net->wb[1], net->wb[2], u.w0p,
                           u.wf[0], u.wf[1], u.wt[0], u.wt[1]);
    // The tensors go out row-major only where the caller can read them (keep): 16 steps
    // with and without these stores, batch 2,048 326 and 312 us, 8,192 658 and 645
    // (4,096, one tile per CU, 418 and 427: no reason to write what nobody reads).
    const unsigned tiles = blocks_for(B, kTrainFT);
    if (apart || full == u.slices) {
        if (keep && apart)
            hipLaunchKernelGGL((k_mlp_train<true, false>), dim3(tiles), dim3(512), 0, stream, io);
        else
            hipLaunchKernelGGL((k_mlp_train<false, false>), dim3(tiles), dim3(512), 0, stream, io);
        hipLaunchKernelGGL(k_mlp_update<false>, dim3(kUpBlocks), dim3(64 * kUpWaves), 0, stream, u);
    } else {
        hipLaunchKernelGGL((k_mlp_train<false, true>), dim3(tiles), dim3(512), 0, stream, io);
        hipLaunchKernelGGL(k_mlp_update<true>, dim3(kUpBlocks), dim3(64 * kUpWaves), 0, stream, u);
    }
    if (keep && !apart) {
        RowMajorArgs r{{io.hT[0], io.hT[1], io.hT[2], io.gT[0], io.gT[1], io.gT[2], io.xT, io.g4T},
                       {io.h_out[0], io.h_out[1], io.h_out[2], io.g_out[0], io.g_out[1], io.g_out[2], io.x_out, io.gout},
                       {256, 256, 256, 256, 256, 256, kFeatLd, 2}, B};
        hipLaunchKernelGGL(k_row_major, dim3(blocks_for(B, 8), 8), dim3(256), 0, stream, r);
    }
    return launched("pn_mlp_train_step");
}

}  // namespace

extern "C" {

pn_status pn_mlp_train_step(pn_mlp* net, const float* feat, const float* label, const float* target,
                            const int32_t* idx, int32_t batch, int32_t step, float lr, float* loss,
                            void* ws, size_t ws_bytes, hipStream_t stream) {
    return train_step(net, feat, label, target, idx, batch, step, lr, loss, ws, ws_bytes, stream, true, true);
}

pn_status pn_mlp_train(pn_mlp* net, int32_t* adam_step, const float* feat, const float* label, const float* target,
                       const int32_t* order, int64_t nbatch, int32_t batch, float lr, float* loss, void* ws,
                       size_t ws_bytes, hipStream_t stream) {
    if (!adam_step || *adam_step < 0 || nbatch < 0 || batch <= 0) return PN_EINVAL;
    if (nbatch > 0 && !order) return PN_EINVAL;
    if ((int64_t)*adam_step + nbatch > 0x7fffffffLL) return PN_EINVAL;
    for (int64_t b = 0; b < nbatch; ++b) {
        const pn_status st = train_step(net, feat, label, target, order + b * batch, batch, *adam_step + 1, lr,
                                        loss, ws, ws_bytes, stream, b == 0, b == nbatch - 1);
        if (st != PN_OK) return st;
        *adam_step += 1;
    }
    return PN_OK;
}

size_t pn_mlp_infer_workspace_size(int64_t chunk) {
    if (chunk <= 0) return 0;
    const size_t C = (size_t)chunk;
    return al(C * kFeatLd * 2) + 3 * al(C * 256 * 2);
}

pn_status pn_mlp_infer(const pn_mlp* net, const float* feat, int64_t n, float* out, int64_t chunk, void* ws,
                       size_t ws_bytes, hipStream_t stream) {
    if (!net_ok(net, false) || n < 0 || chunk <= 0 || chunk > (1 << 26)) return PN_EINVAL;
    if (n == 0) return PN_OK;
    if (!feat || !out) return PN_EINVAL;
    if (!ws || ws_bytes < pn_mlp_infer_workspace_size(chunk)) return PN_ENOWS;
    char* p = static_cast<char*>(ws);
    uint16_t* X = (uint16_t*)p;
    p += al((size_t)chunk * kFeatLd * 2);
    uint16_t* h[3];
    for (int l = 0; l < 3; ++l) { h[l] = (uint16_t*)p; p += al((size_t)chunk * 256 * 2); }
    for (int64_t r0 = 0; r0 < n; r0 += chunk) {
        const int64_t rows = (n - r0) < chunk ? (n - r0) : chunk;
        hipLaunchKernelGGL(k_gather_rows, dim3(blocks_for(rows * kFeatLd, 256)), dim3(256), 0, stream, feat,
                           (const int32_t*)nullptr, rows, r0, X);
        forward(stream, net, rows, X, h[0], h[1], h[2], out + 2 * r0);
    }
    return launched("pn_mlp_infer");
}

pn_status pn_mlp_infer_fused(const pn_mlp* net, const float* feat, int64_t n, float* out, hipStream_t stream) {
    if (!net_ok(net, false) || n < 0) return PN_EINVAL;
    if (n == 0) return PN_OK;
    if (!feat || !out || (reinterpret_cast<uintptr_t>(feat) & 15u) != 0) return PN_EINVAL;
    const int ncu = device_cu_count();
    if (ncu <= 0) {
        pn_detail::set_last_error("pn_mlp_infer_fused", "no device");
        return PN_EDEVICE;
    }
    launch_infer(stream, net, feat, n, out, ncu);
    return launched("pn_mlp_infer_fused");
}

pn_status pn_mlp_features(pn_params params, int64_t n, const double* r0, const double* th1, const double* th2,
                          const double* t_end, double t_end_all, const int32_t* idx, const float* mean,
                          const float* stdv, float* feat, hipStream_t stream) {
    if (n < 0 || !mean || !stdv) return PN_EINVAL;
    const int nnull = (params.beta == nullptr) + (params.chi1 == nullptr) + (params.chi2 == nullptr);
    if (nnull != 0 && nnull != 3) return PN_EINVAL;
    if (!t_end && !(t_end_all > 0.0 && std::isfinite(t_end_all))) return PN_EINVAL;
    for (int c = 0; c < 7; ++c)
        if (!(stdv[c] > 0.0f) || !std::isfinite(stdv[c]) || !std::isfinite(mean[c])) return PN_EINVAL;
    if (n == 0) return PN_OK;
    if (!r0 || !th1 || !th2 || !feat) return PN_EINVAL;
    FeatArgs f;
    f.beta = params.beta; f.chi1 = params.chi1; f.chi2 = params.chi2;
    f.beta0 = params.beta0; f.chi1_0 = params.chi1_0; f.chi2_0 = params.chi2_0;
    f.r0 = r0; f.th1 = th1; f.th2 = th2; f.t_end = t_end; f.t_end_all = t_end_all;
    f.idx = idx; f.n = n; f.feat = feat;
    for (int c = 0; c < 7; ++c) { f.mean[c] = mean[c]; f.stdv[c] = stdv[c]; }
    hipLaunchKernelGGL(k_features, dim3(blocks_for(n, 256)), dim3(256), 0, stream, f);
    return launched("pn_mlp_features");
}

pn_status pn_mlp_targets(const double* fli, const int8_t* label, const double* t_end, double t_end_all, int64_t n,
                         float* lab, float* target, hipStream_t stream) {
    if (n < 0) return PN_EINVAL;
    if (n == 0) return PN_OK;
    if (!fli || !label || !lab || !target) return PN_EINVAL;
    if (!t_end && !(t_end_all > 0.0 && std::isfinite(t_end_all))) return PN_EINVAL;
    hipLaunchKernelGGL(k_targets, dim3(blocks_for(n, 256)), dim3(256), 0, stream, fli, label, t_end, t_end_all, n,
                       lab, target);
    return launched("pn_mlp_targets");
}

pn_status pn_surrogate_gate(const float* out, int64_t n, float margin, double audit_frac, uint64_t seed,
                            int8_t* label, float* fli_pred, int32_t* list, unsigned long long* count,
                            hipStream_t stream) {
    if (n < 0 || !(margin >= 0.0f) || !(audit_frac >= 0.0 && audit_frac <= 1.0)) return PN_EINVAL;
    if (!count) return PN_EINVAL;
    hipLaunchKernelGGL(k_clear_count, dim3(1), dim3(1), 0, stream, count);
    if (n == 0) return launched("pn_surrogate_gate");
    if (!out || !label || !list || n > 0x7fffffffLL) return PN_EINVAL;
    hipLaunchKernelGGL(k_gate, dim3(blocks_for(n, 256)), dim3(256), 0, stream, out, n, margin, audit_frac,
                       (unsigned long long)seed, label, fli_pred, list, count);
    return launched("pn_surrogate_gate");
}

pn_status pn_surrogate_merge(const int32_t* list, int64_t m, const int8_t* integrated, int8_t* label,
                             hipStream_t stream) {
    if (m < 0) return PN_EINVAL;
    if (m == 0) return PN_OK;
    if (!list || !integrated || !label) return PN_EINVAL;
    hipLaunchKernelGGL(k_merge, dim3(blocks_for(m, 256)), dim3(256), 0, stream, list, m, integrated, label);
    return launched("pn_surrogate_merge");
}

pn_status pn_gemm_bf16(int32_t M, int32_t N, int32_t K, const uint16_t* A, int64_t sam, int64_t sak,
                       const uint16_t* B, int64_t sbk, int64_t sbn, const float* bias, int32_t relu,
                       const uint16_t* mask, int64_t ldm, float* Cf, int64_t ldcf, uint16_t* Cb, int64_t ldcb,
                       hipStream_t stream) {
    if (M < 0 || N < 0 || K < 0) return PN_EINVAL;
    if (M == 0 || N == 0) return PN_OK;
    if (!A || !B || (!Cf && !Cb)) return PN_EINVAL;
    if ((Cf && ldcf < N) || (Cb && ldcb < N) || (mask && ldm < N)) return PN_EINVAL;
    gemm(stream, M, N, K, A, sam, sak, B, sbk, sbn, bias, relu, mask, ldm, Cf, ldcf, Cb, ldcb);
    return launched("pn_gemm_bf16");
}

void pn_default_surrogate_cfg(pn_surrogate_cfg* c) {
    if (!c) return;
    c->margin = 0.5f;
    c->audit_frac = 0.01;
    c->seed = 5;
    c->refine_epochs = 40;
    c->refine_batch = 2048;
    c->refine_lr = 5e-4f;
    c->refine_seed = 51;
    c->refine_cosine = 0;
    c->audit_split = 0;
}

// Records of the balanced integrations: min(n, 2^17) slots.  The balanced
// schedule is only taken for at least as many points as the device keeps
// orbit pairs resident, and 2^17 pairs is four wavefronts on every SIMD of
// 256 CUs.
static size_t wrap_region_bytes(int64_t n) {
    const int64_t cap = (int64_t)1 << 17;
    return pn_fli_scan_balanced_workspace_size(n < cap ? n : cap);
}

size_t pn_surrogate_scan_workspace_size(int64_t n, int32_t refine_batch) {
    if (n <= 0 || n > 0x7fffffffLL || refine_batch <= 0) return 0;
    const size_t N = (size_t)n;
    return 2 * al(N * kFeatLd * 4) + al(N * 2 * 4) + 3 * al(N * 4) + al(4 * 8) + al(12 * N * 8) + 4 * al(N * 8) +
           al(N * 8) + al(N) + al(N * 4) + al(N * 8) + 2 * al(N * 4) + al(4) + pn_batch_workspace_size(n) +
           al(wrap_region_bytes(n)) + pn_mlp_train_workspace_size(refine_batch);
}

}  // extern "C"

namespace {

// SplitMix64 stream for the host-side order of the refinement samples.
struct SplitMix {
    uint64_t s;
    uint64_t next() {
        uint64_t x = (s += 0x9e3779b97f4a7c15ull);
        x = (x ^ (x >> 30)) * 0xbf58476d1ce4e5b9ull;
        x = (x ^ (x >> 27)) * 0x94d049bb133111ebull;
        return x ^ (x >> 31);
    }
};

#define PN_TRY(call)                                  \
    do {                                              \
        const pn_status st_ = (call);                 \
        if (st_ != PN_OK) return st_;                 \
    } while (0)

#define PN_HIP(call, what)                                                        \
    do {                                                                          \
        const hipError_t e_ = (call);                                             \
        if (e_ != hipSuccess) {                                                   \
            pn_detail::set_last_error(what, hipGetErrorString(e_));               \
            return PN_EDEVICE;                                                    \
        }                                                                         \
    } while (0)

}  // namespace

extern "C" {

pn_status pn_surrogate_scan(pn_mlp* net, int32_t* adam_step, const pn_model* model, pn_params params,
                            const pn_integrator* integ, const pn_correction* corr, const pn_fli_cfg* fli,
                            int64_t n, const double* r0, const double* p0, const double* th1, const double* ph1,
                            const double* th2, const double* ph2, const double* t_end, double t_end_all,
                            const float* mean, const float* stdv, const pn_surrogate_cfg* cfg, int8_t* label,
                            int32_t* points, int64_t* integrated, pn_surrogate_stats* stats, void* ws,
                            size_t ws_bytes, hipStream_t stream) {
    const char* what = "pn_surrogate_scan";
    if (!cfg || !label || !integrated || n < 0 || n > 0x7fffffffLL) return PN_EINVAL;
    if (!(cfg->margin >= 0.0f) || !(cfg->audit_frac >= 0.0 && cfg->audit_frac <= 1.0)) return PN_EINVAL;
    if (cfg->refine_epochs < 0 || cfg->refine_batch <= 0) return PN_EINVAL;
    if (cfg->refine_cosine != 0 && cfg->refine_cosine != 1) return PN_EINVAL;
    if (cfg->audit_split < 0) return PN_EINVAL;
    if (cfg->refine_epochs > 0 && (!adam_step || *adam_step < 0 || !(cfg->refine_lr > 0.0f))) return PN_EINVAL;
    if (!net_ok(net, cfg->refine_epochs > 0)) return PN_EINVAL;
    if (!r0 || !p0 || !th1 || !ph1 || !th2 || !ph2 || !mean || !stdv) return PN_EINVAL;
    if (!t_end && !(t_end_all > 0.0 && std::isfinite(t_end_all))) return PN_EINVAL;
    for (int c = 0; c < 7; ++c)
        if (!(stdv[c] > 0.0f) || !std::isfinite(stdv[c]) || !std::isfinite(mean[c])) return PN_EINVAL;
    {   // model, parameters, integrator, correction and FLI settings: the scan's own checks, nothing launched
        pn_scan_out so0;
        std::memset(&so0, 0, sizeof(so0));
        if (pn_fli_scan(model, params, integ, corr, fli, 0, nullptr, 0, nullptr, 1.0, &so0, stream) != PN_OK)
            return PN_EINVAL;
    }
    *integrated = 0;
    if (n == 0) return PN_OK;
    if (!ws || ws_bytes < pn_surrogate_scan_workspace_size(n, cfg->refine_batch)) return PN_ENOWS;
    const size_t N = (size_t)n;
    char* p = static_cast<char*>(ws);
    auto take = [&](size_t bytes) { char* q = p; p += al(bytes); return q; };
    float* feat = (float*)take(N * kFeatLd * 4);
    float* featA = (float*)take(N * kFeatLd * 4);
    float* out = (float*)take(N * 2 * 4);
    int32_t* listA = (int32_t*)take(N * 4);
    int32_t* listU = (int32_t*)take(N * 4);
    int32_t* order = (int32_t*)take(N * 4);
    // counts: [0] audit points, [1] uncertain points, [2], [3] orbit-steps
    // integrated by the audit and by the fallback.
    unsigned long long* counts = (unsigned long long*)take(4 * 8);
    double* y0 = (double*)take(12 * N * 8);
    double* gp[4];
    for (int c = 0; c < 4; ++c) gp[c] = (double*)take(N * 8);
    double* sfli = (double*)take(N * 8);
    int8_t* slab = (int8_t*)take(N);
    int32_t* sstat = (int32_t*)take(N * 4);
    int64_t* ssteps = (int64_t*)take(N * 8);
    float* labA = (float*)take(N * 4);
    float* tgtA = (float*)take(N * 4);
    float* loss = (float*)take(4);
    void* bws = take(pn_batch_workspace_size(n));
    const size_t wrap_bytes = wrap_region_bytes(n);
    void* wws = take(wrap_bytes);
    void* tws = take(pn_mlp_train_workspace_size(cfg->refine_batch));
    const bool per_orbit = params.beta != nullptr;

    // Phase timing from events on the stream: ev[0..4] bound the four
    // phases, ev[5..6] and ev[7..8] the scan call of the audit and of the
    // fallback integration.
    hipEvent_t ev[9] = {};
    struct EventGuard {
        hipEvent_t* e;
        ~EventGuard() { for (int k = 0; k < 9; ++k) if (e[k]) (void)hipEventDestroy(e[k]); }
    } guard{ev};
    if (stats) {
        std::memset(stats, 0, sizeof(*stats));
        for (int k = 0; k < 9; ++k) PN_HIP(hipEventCreate(&ev[k]), what);
    }
    auto mark = [&](int k) -> pn_status {
        if (stats) PN_HIP(hipEventRecord(ev[k], stream), what);
        return PN_OK;
    };

    // Integrate the m listed points (phase 0: audit, 1: fallback), labels
    // into slab[0..m), completed steps summed into counts[2 + phase]: points
    // that all end at t_end_all through the balanced scan (which keeps the
    // plain fused scan where that is predicted faster), others with the
    // persistent batch kernel.
    auto integrate = [&](const int32_t* list, int64_t m, int phase) -> pn_status {
        PN_TRY(pn_init_state_gather(model, params, m, list, r0, p0, th1, ph1, th2, ph2, y0, m, stream));
        const unsigned g = blocks_for(m, 256);
        hipLaunchKernelGGL(k_gather_f64, dim3(g), dim3(256), 0, stream, t_end, t_end_all, list, m, gp[3]);
        pn_params q = params;
        if (per_orbit) {
            hipLaunchKernelGGL(k_gather_f64, dim3(g), dim3(256), 0, stream, params.beta, 0.0, list, m, gp[0]);
            hipLaunchKernelGGL(k_gather_f64, dim3(g), dim3(256), 0, stream, params.chi1, 0.0, list, m, gp[1]);
            hipLaunchKernelGGL(k_gather_f64, dim3(g), dim3(256), 0, stream, params.chi2, 0.0, list, m, gp[2]);
            q.beta = gp[0]; q.chi1 = gp[1]; q.chi2 = gp[2];
        }
        PN_TRY(launched(what));
        pn_scan_out so;
        std::memset(&so, 0, sizeof(so));
        so.fli = sfli; so.label = slab; so.status = sstat; so.steps = ssteps;
        int32_t kind = 3, launches = 1;
        bool balanced = false;
        if (t_end == nullptr) {
            int64_t slots = 0;
            int32_t nl = 0;
            PN_TRY(pn_fli_scan_balanced_schedule(integ, corr, m, t_end_all, 0, &slots, nullptr, &nl));
            if (pn_fli_scan_balanced_workspace_size(slots) <= wrap_bytes) {
                balanced = true;
                kind = nl > 0 ? 2 : 1;
                launches = nl > 0 ? nl : 1;
            }
        }
        PN_TRY(mark(5 + 2 * phase));
        if (balanced) {
            PN_TRY(pn_fli_scan_balanced(model, q, integ, corr, fli, m, y0, m, t_end_all, &so, 0, wws, wrap_bytes,
                                        stream));
        } else {
            PN_TRY(pn_batch_scan(model, q, integ, corr, fli, m, y0, m, gp[3], &so, nullptr, bws,
                                 pn_batch_workspace_size(m), stream));
        }
        PN_TRY(mark(6 + 2 * phase));
        hipLaunchKernelGGL(k_sum_steps, dim3(g < 1024 ? g : 1024), dim3(256), 0, stream, ssteps, m,
                           counts + 2 + phase);
        PN_TRY(launched(what));
        if (stats) {
            stats->scan_kernel[phase] = kind;
            stats->scan_launches[phase] = launches;
            stats->points[phase] = m;
        }
        return PN_OK;
    };

    PN_TRY(mark(0));
    // 1. Features of every point; the audit list, by increasing index.  The
    //    list of uncertain points, not yet in use, holds the places of the
    //    workgroups' points (one per kAuditPoints points).
    PN_TRY(pn_mlp_features(params, n, r0, th1, th2, t_end, t_end_all, nullptr, mean, stdv, feat, stream));
    hipLaunchKernelGGL(k_clear_count, dim3(1), dim3(4), 0, stream, counts);
    const unsigned blocks = blocks_for(n, kAuditPoints);
    uint32_t* const first = reinterpret_cast<uint32_t*>(listU);
    hipLaunchKernelGGL(k_audit_count, dim3(blocks), dim3(256), 0, stream, n, cfg->audit_frac,
                       (unsigned long long)cfg->seed, first);
    hipLaunchKernelGGL(k_audit_scan, dim3(1), dim3(1024), 0, stream, first, (int64_t)blocks, counts);
    hipLaunchKernelGGL(k_audit_list, dim3(blocks), dim3(256), 0, stream, n, cfg->audit_frac,
                       (unsigned long long)cfg->seed, first, listA);
    PN_TRY(launched(what));
    unsigned long long cnt = 0;
    PN_HIP(hipMemcpyAsync(&cnt, counts, 8, hipMemcpyDeviceToHost, stream), what);
    PN_HIP(hipStreamSynchronize(stream), what);
    const int64_t ma = (int64_t)cnt;
    // 2. Integrate the audit: all of it, or (audit_split) its first whole
    //    number of scheduling rounds of the batch kernel; the rest of the
    //    audit is then integrated with the uncertain points in step 5, so
    //    that only one of the two integrations ends in a partial round.
    int64_t round = 0;
    if (cfg->audit_split == 1) {
        round = pn_batch_resident_pairs(nullptr);
        if (round <= 0) {
            pn_detail::set_last_error(what, "no device");
            return PN_EDEVICE;
        }
    } else if (cfg->audit_split > 1) {
        round = cfg->audit_split;
    }
    int64_t m1 = ma;
    if (round > 0 && ma >= round) m1 = (ma / round) * round;
    const int64_t m2 = ma - m1;                            // audit points left for step 5
    if (m1 > 0) PN_TRY(integrate(listA, m1, 0));
    PN_TRY(mark(1));
    // 3. Refine the network on the integrated audit points (valid orbits
    //    only), in a SplitMix64-seeded order per epoch.
    if (cfg->refine_epochs > 0 && m1 >= cfg->refine_batch) {
        PN_TRY(pn_mlp_features(params, m1, r0, th1, th2, t_end, t_end_all, listA, mean, stdv, featA, stream));
        if (t_end) {
            PN_TRY(pn_mlp_targets(sfli, slab, gp[3], 0.0, m1, labA, tgtA, stream));
        } else {
            PN_TRY(pn_mlp_targets(sfli, slab, nullptr, t_end_all, m1, labA, tgtA, stream));
        }
        std::vector<int32_t> st((size_t)m1);
        PN_HIP(hipMemcpyAsync(st.data(), sstat, (size_t)m1 * 4, hipMemcpyDeviceToHost, stream), what);
        PN_HIP(hipStreamSynchronize(stream), what);
        std::vector<int32_t> valid;
        valid.reserve((size_t)m1);
        for (int64_t j = 0; j < m1; ++j)
            if ((st[(size_t)j] & 0xFF) == 0) valid.push_back((int32_t)j);
        const int64_t nv = (int64_t)valid.size();
        const int64_t nb = nv / cfg->refine_batch;
        SplitMix rng{cfg->refine_seed};
        std::vector<int32_t> ord(valid);
        // The epochs' orders are drawn on the host in sequence and uploaded in
        // groups, at most as many epochs as the order buffer (n entries) holds:
        // a fifth of them, so that the device waits for the first group only
        // and trains on each while the next is drawn (a draw costs a third of
        // its epoch's training).  2,640 points, 40 epochs: 0.6 ms in one group.
        const int64_t per_copy =
            nv > 0 ? std::max<int64_t>(1, std::min<int64_t>((int64_t)N / nv, (cfg->refine_epochs - 1) / 5 + 1)) : 1;
        // Two host buffers in turn, each refilled once its copy is done; they
        // outlive every copy, also where a call in between fails.
        std::vector<int32_t> orders[2];
        struct Copies {
            hipEvent_t done[2] = {};
            bool pending[2] = {};
            ~Copies() {
                for (int c = 0; c < 2; ++c) {
                    if (pending[c]) (void)hipEventSynchronize(done[c]);
                    if (done[c]) (void)hipEventDestroy(done[c]);
                }
            }
        } copies;
        for (int c = 0; c < 2; ++c) PN_HIP(hipEventCreateWithFlags(&copies.done[c], hipEventDisableTiming), what);
        int buf = 0;
        for (int32_t e0 = 0; e0 < cfg->refine_epochs && nb > 0; e0 += (int32_t)per_copy, buf ^= 1) {
            const int32_t ne = (int32_t)std::min<int64_t>(per_copy, cfg->refine_epochs - e0);
            if (copies.pending[buf]) PN_HIP(hipEventSynchronize(copies.done[buf]), what);
            std::vector<int32_t>& o = orders[buf];
            o.resize((size_t)ne * (size_t)nv);
            for (int32_t k = 0; k < ne; ++k) {
                for (size_t q = ord.size(); q > 1; --q) {      // Fisher-Yates
                    const size_t r = (size_t)(rng.next() % q);
                    std::swap(ord[q - 1], ord[r]);
                }
                std::copy(ord.begin(), ord.end(), o.begin() + (size_t)k * (size_t)nv);
            }
            // In stream order: the buffer's earlier group has been trained on.
            PN_HIP(hipMemcpyAsync(order, o.data(), o.size() * 4, hipMemcpyHostToDevice, stream), what);
            PN_HIP(hipEventRecord(copies.done[buf], stream), what);
            copies.pending[buf] = true;
            for (int32_t k = 0; k < ne; ++k) {
                const int32_t e = e0 + k;
                // The weights' other layouts are formed before the first
                // refinement step; each step's update keeps them current.
                const float lr_e = cfg->refine_cosine
                                       ? cfg->refine_lr * 0.5f *
                                             (1.0f + cosf(3.14159265358979f * e / cfg->refine_epochs))
                                       : cfg->refine_lr;
                for (int64_t b = 0; b < nb; ++b) {
                    *adam_step += 1;
                    PN_TRY(train_step(net, featA, labA, tgtA, order + (size_t)k * nv + b * cfg->refine_batch,
                                      cfg->refine_batch, *adam_step, lr_e, loss, tws,
                                      pn_mlp_train_workspace_size(cfg->refine_batch), stream,
                                      e == 0 && b == 0, false));
                }
            }
        }
    }
    PN_TRY(mark(2));
    // 4. Inference and the gate of the uncertain, not audited points.
    PN_TRY(pn_mlp_infer_fused(net, feat, n, out, stream));
    hipLaunchKernelGGL(k_gate_uncertain, dim3(blocks_for(n, 256)), dim3(256), 0, stream, out, n, cfg->margin,
                       cfg->audit_frac, (unsigned long long)cfg->seed, label, listU, counts + 1);
    PN_TRY(launched(what));
    // The integrated audit labels (in slab) are merged before the next scan
    // reuses it.
    if (m1 > 0) PN_TRY(pn_surrogate_merge(listA, m1, slab, label, stream));
    PN_HIP(hipMemcpyAsync(&cnt, counts + 1, 8, hipMemcpyDeviceToHost, stream), what);
    PN_HIP(hipStreamSynchronize(stream), what);
    const int64_t mu = (int64_t)cnt;
    PN_TRY(mark(3));
    // 5. Integrate the rest of the audit and the uncertain points in one
    //    batch (the training order buffer holds the joined list); their
    //    labels replace the network's.
    if (m2 + mu > 0) {
        const int32_t* list5 = listU;
        if (m2 > 0) {
            PN_HIP(hipMemcpyAsync(order, listA + m1, (size_t)m2 * 4, hipMemcpyDeviceToDevice, stream), what);
            if (mu > 0)
                PN_HIP(hipMemcpyAsync(order + m2, listU, (size_t)mu * 4, hipMemcpyDeviceToDevice, stream), what);
            list5 = order;
        }
        PN_TRY(integrate(list5, m2 + mu, 1));
        PN_TRY(pn_surrogate_merge(list5, m2 + mu, slab, label, stream));
    }
    if (points) {
        if (ma > 0) PN_HIP(hipMemcpyAsync(points, listA, (size_t)ma * 4, hipMemcpyDeviceToDevice, stream), what);
        if (mu > 0) PN_HIP(hipMemcpyAsync(points + ma, listU, (size_t)mu * 4, hipMemcpyDeviceToDevice, stream), what);
    }
    PN_TRY(mark(4));
    if (stats) {
        unsigned long long steps2[2] = {0, 0};
        PN_HIP(hipMemcpyAsync(steps2, counts + 2, 16, hipMemcpyDeviceToHost, stream), what);
        PN_HIP(hipStreamSynchronize(stream), what);
        for (int k = 0; k < 4; ++k) PN_HIP(hipEventElapsedTime(&stats->phase_ms[k], ev[k], ev[k + 1]), what);
        for (int k = 0; k < 2; ++k) {
            if (stats->scan_launches[k] > 0)
                PN_HIP(hipEventElapsedTime(&stats->scan_ms[k], ev[5 + 2 * k], ev[6 + 2 * k]), what);
            stats->orbit_steps[k] = (int64_t)steps2[k];
        }
    }
    *integrated = ma + mu;
    return PN_OK;
}

}  // extern "C"
