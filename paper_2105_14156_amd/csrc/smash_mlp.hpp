// smash_mlp.hpp -- the learned row-size predictor: per-row features, MLP
// inference, and the training kernels (forward, backward, Adam).
//
// The network maps six per-row features of C = A * B to log2(1 + nnz(C_i)):
// 6 -> 64 -> 64 -> 1, ReLU hidden layers, FP32, parameters packed as
// W1[64][6], b1[64], W2[64][64], b2[64], w3[64], b3.  A predicted capacity
// per row lets the fused pass size its LDS tables without a symbolic pass.
// Training minimises the mean squared error with Adam (Kingma and Ba 2015)
// on batches of rows whose exact counts come from the symbolic phase.
// Reductions over a batch use fixed orders (no atomics), so training is
// deterministic.  Predictions for many rows run on the FP32 matrix
// instructions (k_mlp_rows), and training's FP64 gradient sums on the FP64 ones
// (k_mlp_step).  The capacities of the fused pass are plain FMA (k_mlp_predict):
// only rows above the LDS limit are asked about, often one among the rows of a
// wave, too few for a matrix tile.
#pragma once

#include <hip/hip_runtime.h>

#include "smash_kernels.hpp"

namespace smash {

constexpr int kFeat = 6;
constexpr int kHid = 64;
constexpr int kOW1 = 0;
constexpr int kOB1 = kOW1 + kHid * kFeat;
constexpr int kOW2 = kOB1 + kHid;
constexpr int kOB2 = kOW2 + kHid * kHid;
constexpr int kOW3 = kOB2 + kHid;
constexpr int kOB3 = kOW3 + kHid;
constexpr int kParams = kOB3 + 1;     // 4673

// Features of each row i: log2(1 + x) of nnz(A_i), the products ub_i, max_k
// nnz(B_k), min_k nnz(B_k), min(ub_i, cols) and sum_k nnz(B_k)^2 / ub_i, from
// the sums of the row analysis (for_rows; a wave per row took 62 us where this
// takes 21: 131072 rows, RMAT scale 17, edge factor 8).
__global__ __launch_bounds__(kRowThreads) void k_features(int m, int ncols, const int *__restrict__ Arp,
                                                          const int *__restrict__ Acol,
                                                          const int *__restrict__ Brp, float *__restrict__ feats)
{
    for_rows<true>(m, Arp, Acol, Brp, [&](int row, int sl, int e0, int e1, const RowPart &r) {
        if (sl < kFeat)
            feats[(long long)row * kFeat + sl] = row_feature(sl, e1 - e0, r.ub, r.sq, r.mx, r.mn, ncols);
    });
}

__device__ __forceinline__ void load_params(float *s_w, const float *__restrict__ theta)
{
    for (int t = threadIdx.x; t < kParams; t += blockDim.x) s_w[t] = theta[t];
}

// Network output for one standardized feature vector.
__device__ __forceinline__ float mlp_eval(const float *s_w, const float x[kFeat])
{
    float h1[kHid];
#pragma unroll
    for (int i = 0; i < kHid; ++i) {
        float z = s_w[kOB1 + i];
#pragma unroll
        for (int f = 0; f < kFeat; ++f) z = fmaf(s_w[kOW1 + i * kFeat + f], x[f], z);
        h1[i] = z > 0.f ? z : 0.f;
    }
    float y = s_w[kOB3];
    for (int j = 0; j < kHid; ++j) {
        float z = s_w[kOB2 + j];
#pragma unroll
        for (int i = 0; i < kHid; ++i) z = fmaf(s_w[kOW2 + j * kHid + i], h1[i], z);
        y = fmaf(s_w[kOW3 + j], z > 0.f ? z : 0.f, y);
    }
    return y;
}

// Capacity of a row from the network's output y: clamp(ceil(2^(y + delta)
// - 1), max(maxb, 1), min(ub, cols)), 0 for a row without products.
__device__ __forceinline__ int predicted_capacity(float y, float delta, long long u, int maxb_i, int ncols)
{
    if (u <= 0) return 0;
    const long long hi = u < ncols ? u : ncols;
    const long long lo = maxb_i > 1 ? maxb_i : 1;
    float p = exp2f(y + delta) - 1.f;
    long long c = p < 1.f ? 1 : (p > 2.0e9f ? 2000000000LL : (long long)ceilf(p));
    c = c < lo ? lo : c;
    c = c > hi ? hi : c;
    return (int)c;
}

// A wave whose candidate rows are at most this many evaluates them one at a
// time, a hidden unit per lane, instead of a row per lane.
constexpr int kMlpSparseRows = 8;

// Predicted capacities (predicted_capacity): the network is evaluated only
// for rows whose exact bound min(ub, cols) exceeds only_above (the rows a
// prediction can move into the LDS tables); the others get the bound
// itself, and a block without such rows loads no weights.  A wave with many
// candidate rows evaluates a row per lane; a wave with few (where the
// candidates are rare, most lanes of a row-per-lane wave would idle through
// the whole network) takes them one by one with lane j computing hidden
// unit j of both layers, reading the other units' values with v_readlane.
// Both forms add in the same order, so a row's result does not depend on
// which form evaluated it.
__global__ __launch_bounds__(256) void k_mlp_predict(int m, int ncols, const float *__restrict__ feats,
                                                     const float *__restrict__ theta, const float *__restrict__ ms,
                                                     float delta, const long long *__restrict__ ub,
                                                     const int *__restrict__ maxb, int *__restrict__ cap_out,
                                                     int only_above)
{
    static_assert(kHid == kWave, "one hidden unit per lane");
    __shared__ float s_w[kParams];
    __shared__ float s_ms[2 * kFeat];
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    const int lane = threadIdx.x & (kWave - 1);
    const bool live = i < m;
    const long long ub_i = live ? ub[i] : 0;
    const long long bound = ub_i < ncols ? ub_i : ncols;
    const bool cand = live && bound > only_above;
    if (!__syncthreads_or(cand)) {
        if (live) cap_out[i] = (int)bound;
        return;
    }
    load_params(s_w, theta);
    if (threadIdx.x < 2 * kFeat) s_ms[threadIdx.x] = ms[threadIdx.x];
    __syncthreads();
    if (live && !cand) cap_out[i] = (int)bound;
    const unsigned long long cm = __builtin_amdgcn_ballot_w64(cand);
    if (__popcll(cm) > kMlpSparseRows) {
        if (!cand) return;
        float x[kFeat];
#pragma unroll
        for (int f = 0; f < kFeat; ++f) x[f] = (feats[(long long)i * kFeat + f] - s_ms[f]) / s_ms[kFeat + f];
        const float y = mlp_eval(s_w, x);
        cap_out[i] = predicted_capacity(y, delta, ub[i], maxb[i], ncols);
        return;
    }
    if (!cm) return;
    // few candidates: lane j is hidden unit j; its rows of W1 and W2 are
    // read once from the parameters in global memory (a row of W2 in LDS
    // lies in one bank for every lane)
    float w1[kFeat], w2[kHid];
#pragma unroll
    for (int f = 0; f < kFeat; ++f) w1[f] = theta[kOW1 + lane * kFeat + f];
#pragma unroll
    for (int q = 0; q < kHid; ++q) w2[q] = theta[kOW2 + lane * kHid + q];
    const float b1 = s_w[kOB1 + lane], b2 = s_w[kOB2 + lane];
    const int row0 = i - lane;
    for (unsigned long long mm = cm; mm; mm &= mm - 1) {
        const int l = __ffsll((long long)mm) - 1;
        const int r = row0 + l;
        float x[kFeat];
#pragma unroll
        for (int f = 0; f < kFeat; ++f) x[f] = (feats[(long long)r * kFeat + f] - s_ms[f]) / s_ms[kFeat + f];
        float z = b1;
#pragma unroll
        for (int f = 0; f < kFeat; ++f) z = fmaf(w1[f], x[f], z);
        const float h1 = z > 0.f ? z : 0.f;
        float z2 = b2;
#pragma unroll
        for (int q = 0; q < kHid; ++q)
            z2 = fmaf(w2[q], __int_as_float(__builtin_amdgcn_readlane(__float_as_int(h1), q)), z2);
        const float h2 = z2 > 0.f ? z2 : 0.f;
        float y = s_w[kOB3];
#pragma unroll
        for (int q = 0; q < kHid; ++q)
            y = fmaf(s_w[kOW3 + q], __int_as_float(__builtin_amdgcn_readlane(__float_as_int(h2), q)), y);
        if (lane == l) cap_out[r] = predicted_capacity(y, delta, ub[r], maxb[r], ncols);
    }
}

// Inference for every row (smash_mlp_predict): 32 rows per wave and step on
// V_MFMA_F32_32X32X2 (D += A B: lane l gives A[l % 32][k] and B[k][l % 32] with
// k = l / 32, and holds rows 8 (r / 4) + 4 (l / 32) + r % 4, r = 0..15, column
// l % 32 of D).  Units are rows and samples columns of D, so a layer's output
// registers are the next one's B operands as they are: step r contracts the
// two units that register r holds in the two half-waves, and the weights are
// loaded in that order.  They stay in registers; nothing else touches LDS.
// Bound by the matrix unit (70 instructions of 64 cycles per 32 rows) and the
// weights' first load: features and prediction of 131072 rows take 48 us with
// their launches, 58 where a lane took a row with a fused multiply-add per
// weight.  FP32 sums, in another order than there (error against 64 bits
// 7e-8 of the largest output, 1.1e-7 there).
constexpr int kMlpRows = 32;

typedef float mlp_f32x16 __attribute__((ext_vector_type(16)));

__global__ __launch_bounds__(256, 2) void k_mlp_rows(int m, const float *__restrict__ feats,
                                                     const float *__restrict__ theta, const float *__restrict__ ms,
                                                     float *__restrict__ yhat)
{
    constexpr int LD = kHid + 1;
    __shared__ float s_w2[kHid * LD];
    const int lane = lane_id(), s = lane & 31, h = lane >> 5;
    for (int t = threadIdx.x; t < kHid * kHid; t += 256) s_w2[t / kHid * LD + t % kHid] = theta[kOW2 + t];
    __syncthreads();
    float w1[2][3], w2[2][2][16];
#pragma unroll
    for (int i = 0; i < 2; ++i) {
#pragma unroll
        for (int t = 0; t < 3; ++t) w1[i][t] = theta[kOW1 + (i * 32 + s) * kFeat + 2 * t + h];
    }
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int r = 0; r < 16; ++r)
                w2[j][i][r] = s_w2[(j * 32 + s) * LD + i * 32 + 8 * (r >> 2) + 4 * h + (r & 3)];
    float mean[3], dev[3];
#pragma unroll
    for (int t = 0; t < 3; ++t) {
        mean[t] = ms[2 * t + h];
        dev[t] = ms[kFeat + 2 * t + h];
    }
    mlp_f32x16 b1[2], b2[2], w3[2];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            const int u = i * 32 + 8 * (r >> 2) + 4 * h + (r & 3);
            b1[i][r] = theta[kOB1 + u];
            b2[i][r] = theta[kOB2 + u];
            w3[i][r] = theta[kOW3 + u];
        }
    const int tiles = (int)(((long long)m + kMlpRows - 1) / kMlpRows);
    for (int tile = blockIdx.x * 4 + threadIdx.x / kWave; tile < tiles; tile += gridDim.x * 4) {
        const unsigned row = (unsigned)tile * kMlpRows + s;
        mlp_f32x16 z1[2] = {b1[0], b1[1]}, z2[2] = {b2[0], b2[1]};
#pragma unroll
        for (int t = 0; t < 3; ++t) {
            const float x = row < (unsigned)m ? (feats[(long long)row * kFeat + 2 * t + h] - mean[t]) / dev[t] : 0.f;
#pragma unroll
            for (int i = 0; i < 2; ++i) z1[i] = __builtin_amdgcn_mfma_f32_32x32x2f32(w1[i][t], x, z1[i], 0, 0, 0);
        }
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const float a = z1[i][r] > 0.f ? z1[i][r] : 0.f;
#pragma unroll
                for (int j = 0; j < 2; ++j)
                    z2[j] = __builtin_amdgcn_mfma_f32_32x32x2f32(w2[j][i][r], a, z2[j], 0, 0, 0);
            }
        float y = 0.f;
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) y = fmaf(w3[j][r], z2[j][r] > 0.f ? z2[j][r] : 0.f, y);
        y += __shfl_xor(y, 32, kWave);
        if (h == 0 && row < (unsigned)m) yhat[row] = y + theta[kOB3];
    }
}

// ------------------------------------------------------------ training

// One training step is two launches: k_mlp_step takes the batch forward and
// backward in tiles of 64 samples and leaves one partial gradient per block;
// k_mlp_adam (or k_mlp_grad) adds the partials in block order and updates.
// Everything a tile computes stays in registers and LDS.  At batch 4096 the
// step is bound by latency (18M multiply-adds on 64 of 256 CUs): five separate
// kernels through global activations took 371 us a step, 292 of them in the
// 64 x 64 x batch contraction dW2 on 64 blocks of strided loads; as two
// launches with that contraction on the FP64 matrix instruction a step takes
// 32 us (23 forward and backward, 6 sums and update).
constexpr int kTrainTile = 64;        // samples per tile: one per lane
constexpr int kTrainThreads = 256;    // four waves: 16 hidden units each
constexpr int kTrainMaxBlocks = 256;  // partial gradients at most (one block per CU)
constexpr int kTrainLd = kTrainTile + 4;

typedef double mlp_f64x4 __attribute__((ext_vector_type(4)));

// The gradient sums use V_MFMA_F64_16X16X4 (D += A B): lane l gives A[l % 16][k]
// and B[k][l % 16] with k = l / 16, and holds rows 4 r + l / 16 (r = 0..3),
// column l % 16 of D.  Products of two floats are exact in FP64.  Rows of the
// LDS arrays are padded to 68 floats, so that those reads touch every bank
// once and float4 reads stay aligned.
// Forward and backward of the batch idx[0, n): block b takes tiles b, b +
// gridDim.x, ... and writes its sums of the gradient to part[b] (FP64) and of
// the squared errors to sse_part[b].  The two 64 x 64 x 64 products of a tile
// (z2 = W2 h1 and W2^T dz2) are register tiles of 4 units x 4 samples per
// thread, weights and activations read from LDS as float4; loops stay rolled,
// since straight-line code run once per launch is bound by instruction
// fetches (weights through scalar loads in unrolled code: 44 us a launch at
// batch 4096, 23 us so).  Every unit adds its inputs in the order of
// mlp_eval.  Gradient sums are FP64 in a fixed order (no atomics), so
// training is deterministic.
__global__ __launch_bounds__(kTrainThreads) void k_mlp_step(int n, const int *__restrict__ idx,
                                                            const float *__restrict__ feats,
                                                            const float *__restrict__ y, const float *__restrict__ ms,
                                                            const float *__restrict__ theta, double *__restrict__ part,
                                                            double *__restrict__ sse_part)
{
    static_assert(kTrainTile == kWave && kTrainThreads == 4 * kWave && kHid == 64, "tile shape");
    constexpr int U = kHid / 4;         // hidden units per wave
    __shared__ __align__(16) float s_w[kParams];
    __shared__ __align__(16) float s_h1[kHid * kTrainLd], s_h2[kHid * kTrainLd];
    __shared__ __align__(16) float s_dz2[kHid * kTrainLd], s_dz1[kHid * kTrainLd];
    __shared__ float s_x[16 * kTrainLd];    // rows 0..5 the inputs, row 6 ones, row 7 dL/dy, the others zero
    const int lane = lane_id(), u0 = (int)threadIdx.x / kWave * U;
    const int tu = (int)threadIdx.x / 16 * 4, ts = (int)threadIdx.x % 16 * 4;   // this thread's 4 x 4 tile
    load_params(s_w, theta);
    for (int t = threadIdx.x; t < 16 * kTrainLd; t += kTrainThreads) s_x[t] = t / kTrainLd == kFeat ? 1.f : 0.f;
    mlp_f64x4 gw2[4] = {}, gin = {}, gout = {}, gb2 = {};
    double se = 0.0, gb3 = 0.0;
    for (int tile = blockIdx.x; tile < (n + kTrainTile - 1) / kTrainTile; tile += gridDim.x) {
        const int s = tile * kTrainTile + lane;
        const bool live = s < n;
        const long long r = live ? idx[s] : 0;
        float x[kFeat];
#pragma unroll
        for (int f = 0; f < kFeat; ++f) x[f] = live ? (feats[r * kFeat + f] - ms[f]) / ms[kFeat + f] : 0.f;
        const float target = live ? y[r] : 0.f;
        __syncthreads();                    // weights in; the last tile's sums are done with the arrays
#pragma unroll 4
        for (int i = u0; i < u0 + U; ++i) {
            float z = s_w[kOB1 + i];
#pragma unroll
            for (int f = 0; f < kFeat; ++f) z = fmaf(s_w[kOW1 + i * kFeat + f], x[f], z);
            s_h1[i * kTrainLd + lane] = live && z > 0.f ? z : 0.f;
        }
        __syncthreads();
        float acc[4][4];
#pragma unroll
        for (int u = 0; u < 4; ++u)
#pragma unroll
            for (int q = 0; q < 4; ++q) acc[u][q] = s_w[kOB2 + tu + u];
#pragma unroll 1
        for (int i = 0; i < kHid; i += 4) {
            float4 w[4], h[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) w[u] = *(const float4 *)&s_w[kOW2 + (tu + u) * kHid + i];
#pragma unroll
            for (int k = 0; k < 4; ++k) h[k] = *(const float4 *)&s_h1[(i + k) * kTrainLd + ts];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const float wk[4] = {w[u].x, w[u].y, w[u].z, w[u].w};
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    acc[u][0] = fmaf(wk[k], h[k].x, acc[u][0]);
                    acc[u][1] = fmaf(wk[k], h[k].y, acc[u][1]);
                    acc[u][2] = fmaf(wk[k], h[k].z, acc[u][2]);
                    acc[u][3] = fmaf(wk[k], h[k].w, acc[u][3]);
                }
            }
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            float h[4];
#pragma unroll
            for (int q = 0; q < 4; ++q)
                h[q] = tile * kTrainTile + ts + q < n && acc[u][q] > 0.f ? acc[u][q] : 0.f;
            *(float4 *)&s_h2[(tu + u) * kTrainLd + ts] = make_float4(h[0], h[1], h[2], h[3]);
        }
        __syncthreads();
        float yh = s_w[kOB3];
#pragma unroll 16
        for (int j = 0; j < kHid; ++j) yh = fmaf(s_w[kOW3 + j], s_h2[j * kTrainLd + lane], yh);
        const float res = yh - target;
        const float dy = live ? 2.f * res / (float)n : 0.f;
        if (u0 == 0) {
            se += live ? (double)res * (double)res : 0.0;
            gb3 += (double)dy;
#pragma unroll
            for (int f = 0; f < kFeat; ++f) s_x[f * kTrainLd + lane] = x[f];
            s_x[(kFeat + 1) * kTrainLd + lane] = dy;
        }
#pragma unroll 4
        for (int j = u0; j < u0 + U; ++j)
            s_dz2[j * kTrainLd + lane] = s_h2[j * kTrainLd + lane] > 0.f ? dy * s_w[kOW3 + j] : 0.f;
        __syncthreads();
        // back through W2: dz1_i = (sum_j W2[j][i] dz2_j) [h1_i > 0]
#pragma unroll
        for (int u = 0; u < 4; ++u)
#pragma unroll
            for (int q = 0; q < 4; ++q) acc[u][q] = 0.f;
#pragma unroll 4
        for (int j = 0; j < kHid; ++j) {
            const float4 w = *(const float4 *)&s_w[kOW2 + j * kHid + tu];
            const float4 d = *(const float4 *)&s_dz2[j * kTrainLd + ts];
            const float wu[4] = {w.x, w.y, w.z, w.w};
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                acc[u][0] = fmaf(wu[u], d.x, acc[u][0]);
                acc[u][1] = fmaf(wu[u], d.y, acc[u][1]);
                acc[u][2] = fmaf(wu[u], d.z, acc[u][2]);
                acc[u][3] = fmaf(wu[u], d.w, acc[u][3]);
            }
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const float4 h = *(const float4 *)&s_h1[(tu + u) * kTrainLd + ts];
            *(float4 *)&s_dz1[(tu + u) * kTrainLd + ts] =
                make_float4(h.x > 0.f ? acc[u][0] : 0.f, h.y > 0.f ? acc[u][1] : 0.f, h.z > 0.f ? acc[u][2] : 0.f,
                            h.w > 0.f ? acc[u][3] : 0.f);
        }
        __syncthreads();
        // gradient sums over the tile's samples: dW2 (16 x 64 per wave), db2
        // (against the row of ones), dW1 and db1 (inputs and ones), dw3
#pragma unroll 2
        for (int t = 0; t < kTrainTile / 4; ++t) {
            const int at = (lane & 15) * kTrainLd + (lane >> 4) + 4 * t;
            const double d2 = (double)s_dz2[u0 * kTrainLd + at], xx = (double)s_x[at];
#pragma unroll
            for (int c = 0; c < 4; ++c)
                gw2[c] = __builtin_amdgcn_mfma_f64_16x16x4f64(d2, (double)s_h1[c * 16 * kTrainLd + at], gw2[c], 0, 0, 0);
            gb2 = __builtin_amdgcn_mfma_f64_16x16x4f64(d2, xx, gb2, 0, 0, 0);
            gin = __builtin_amdgcn_mfma_f64_16x16x4f64((double)s_dz1[u0 * kTrainLd + at], xx, gin, 0, 0, 0);
            gout = __builtin_amdgcn_mfma_f64_16x16x4f64((double)s_h2[u0 * kTrainLd + at], xx, gout, 0, 0, 0);
        }
    }
    double *o = part + (long long)blockIdx.x * kParams;
    const int c = lane & 15;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const int u = u0 + 4 * q + (lane >> 4);
#pragma unroll
        for (int t = 0; t < 4; ++t) o[kOW2 + u * kHid + t * 16 + c] = gw2[t][q];
        if (c < kFeat) o[kOW1 + u * kFeat + c] = gin[q];
        if (c == kFeat) {
            o[kOB1 + u] = gin[q];
            o[kOB2 + u] = gb2[q];
        }
        if (c == kFeat + 1) o[kOW3 + u] = gout[q];
    }
    if (u0 == 0) {
        se = wave_sum(se);
        gb3 = wave_sum(gb3);
        if (lane == 0) {
            o[kOB3] = gb3;
            sse_part[blockIdx.x] = se;
        }
    }
}

// Gradient of parameter p: the blocks' partial sums in order.
__device__ __forceinline__ float mlp_grad_sum(int nb, int p, const double *__restrict__ part)
{
    double g = 0.0;
#pragma unroll 16
    for (int b = 0; b < nb; ++b) g += part[(long long)b * kParams + p];
    return (float)g;
}

__global__ __launch_bounds__(kWave) void k_mlp_grad(int nb, const double *__restrict__ part, float *__restrict__ grad)
{
    const int p = blockIdx.x * kWave + threadIdx.x;
    if (p < kParams) grad[p] = mlp_grad_sum(nb, p, part);
}

// Adam update of every parameter from the step's partial gradients (t counts
// steps from 1).
__global__ __launch_bounds__(kWave) void k_mlp_adam(int nb, const double *__restrict__ part, float *__restrict__ theta,
                                                    float *__restrict__ mom, float *__restrict__ vel, int t, float lr,
                                                    float b1, float b2, float eps)
{
    const int p = blockIdx.x * kWave + threadIdx.x;
    if (p >= kParams) return;
    const float g = mlp_grad_sum(nb, p, part);
    const float m = b1 * mom[p] + (1.f - b1) * g;
    const float v = b2 * vel[p] + (1.f - b2) * g * g;
    mom[p] = m;
    vel[p] = v;
    const float mh = m / (1.f - powf(b1, (float)t));
    const float vh = v / (1.f - powf(b2, (float)t));
    theta[p] -= lr * mh / (sqrtf(vh) + eps);
}

}  // namespace smash
