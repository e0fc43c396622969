// Learned closure kernels: per-element P1 moments, network inputs, and a
// small fully connected network (120 -> 64 -> 64 -> 20, tanh) with its
// forward pass, hand-derived backward pass and Adam update.
//
// The closure adds to an order-1 residual the P1 part of the difference
// between the filtered high-order residual and the order-1 residual of the
// filtered state, as predicted from the element's and its face neighbours'
// P1 moments.  Parameter layout: W1 [64][120], b1 [64], W2 [64][64], b2 [64],
// W3 [20][64], b3 [20] (row-major, in this order).
#include <hip/hip_runtime.h>

#include <cmath>
#include <type_traits>

#include "fr_device.hpp"

namespace frd {

namespace {

constexpr int OW1 = 0, OB1 = OW1 + MLP_H * MLP_IN, OW2 = OB1 + MLP_H, OB2 = OW2 + MLP_H * MLP_H;
constexpr int OW3 = OB2 + MLP_H, OB3 = OW3 + MLP_OUT * MLP_H;
static_assert(OB3 + MLP_OUT == MLP_NPARAM, "parameter layout");

// Weight read: FP32 master copy, or its BF16 rounding (stored as the high
// half of the FP32 bit pattern).
template <bool BF16W>
__device__ __forceinline__ float wt(const float *p, const uint16_t *pb, int i) {
    if constexpr (BF16W)
        return __builtin_bit_cast(float, uint32_t(pb[i]) << 16);
    else
        return p[i];
}

// moments mom[g * rs + (v * 4 + a) * cs] = sum_i Mom[a][i] U[i][v][e], g = goff + e
// (element-major rs = 20, cs = 1, or feature-major rs = 1, cs = n_total); of
// U - B when B is given; targets then normalised (m - mu_y) / s_y if ystats
template <typename T>
__global__ __launch_bounds__(256) void moments_kernel(const T *__restrict__ U, const T *__restrict__ B,
                                                      int64_t ld, int64_t nelem, int nu,
                                                      const float *__restrict__ Mom,
                                                      float *__restrict__ mom, int64_t goff, int64_t rs,
                                                      int64_t cs, const float *__restrict__ ystats) {
    const int64_t e = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
    if (e >= nelem) return;
    float m[20];
#pragma unroll
    for (int q = 0; q < 20; ++q) m[q] = 0;
    for (int i = 0; i < nu; ++i)
#pragma unroll
        for (int v = 0; v < 5; ++v) {
            const int64_t o = (int64_t(i) * 5 + v) * ld + e;
            const float u = B ? float(U[o] - B[o]) : float(U[o]);
#pragma unroll
            for (int a = 0; a < 4; ++a) m[v * 4 + a] += Mom[a * nu + i] * u;
        }
    float *out = mom + (goff + e) * rs;
#pragma unroll
    for (int q = 0; q < 20; ++q) out[q * cs] = ystats ? (m[q] - ystats[q]) / ystats[MLP_OUT + q] : m[q];
}

// inputs x[g][0..119]: own moments, then the neighbours' across faces 0..4
// (zeros where there is no such face), normalised (x - mu) / s if stats.
// Moments at mom[g * rs + q * cs], inputs at feat[g * frs + k * fcs].
// A thread takes one element and one of the six sources, blockIdx.y, with its
// twenty loads in flight together: a thread that walked all 120 inputs waited
// for a gather and a division each time (129,024 elements, 62 MB written:
// 45 -> 25 us).
__global__ __launch_bounds__(256) void features_kernel(const float *__restrict__ mom, int64_t rs, int64_t cs,
                                                       const int32_t *__restrict__ nb,
                                                       int64_t ntot,
                                                       const float *__restrict__ stats,
                                                       float *__restrict__ feat, int64_t frs, int64_t fcs) {
    const int64_t g = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
    if (g >= ntot) return;
    const int b = blockIdx.y;
    const int64_t src = b == 0 ? g : nb[g * 5 + b - 1];
    float *out = feat + g * frs + b * 20 * fcs;
    const float *in = mom + (src >= 0 ? src : g) * rs;
    float v[20];
#pragma unroll
    for (int q = 0; q < 20; ++q) v[q] = in[q * cs];
#pragma unroll
    for (int q = 0; q < 20; ++q) {
        float x = src >= 0 ? v[q] : 0.0f;
        if (stats) x = (x - stats[b * 20 + q]) / stats[MLP_IN + b * 20 + q];
        out[q * fcs] = x;
    }
}

typedef float f32x4 __attribute__((ext_vector_type(4)));

// tanh x = 1 - 2 / (1 + e^(2x)) with the hardware base-2 exponential and
// reciprocal: absolute error below 1e-6 over the whole line (e^(2x)
// overflowing to infinity gives 1, underflowing to 0 gives -1)
__device__ __forceinline__ float fast_tanh(float x) {
    const float e = __builtin_amdgcn_exp2f(x * 2.8853900817779268f);   // 2 / ln 2
    return 1.0f - 2.0f * __builtin_amdgcn_rcpf(1.0f + e);
}

// x unchanged but opaque to the optimiser, so that a value loaded ahead of
// a loop stays a separate register set (see the operator-product kernels)
__device__ __forceinline__ float opaque(float x) {
    asm volatile("" : "+v"(x));
    return x;
}

// The network's forward pass on the FP32 matrix cores: one wavefront per 32
// samples, eight per workgroup (two per SIMD).  The workgroup stages the weights (FP32, or
// their BF16 rounding widened to FP32) in LDS.  Each layer is a product of
// 16 x 16 x 4 steps with the samples as rows (A: inputs or activations, lane
// l holding sample l % 16 of a 16-row block at K index l / 16) and the
// transposed weights as B; all output blocks of a layer are accumulated
// together (16 independent accumulators), then bias and tanh are applied on
// the accumulators and the activations go to the wavefront's LDS rows as the
// next layer's A operand.  Inputs at X[s * xrs + k * xcs], outputs at
// Y[s * yrs + o * ycs] (sample-major or feature-major).
constexpr int FWD_HP = MLP_H + 1;                 // padded activation row (no bank conflicts)
constexpr int FWD_WAVES = 8, FWD_MS = 2;          // 8 wavefronts of 32 samples per workgroup
constexpr int FWD_TILE = FWD_WAVES * FWD_MS * 16;
template <bool BF16W>
__global__ __launch_bounds__(512) void mlp_forward_mfma_kernel(const float *__restrict__ P,
                                                               const uint16_t *__restrict__ Pb,
                                                               const float *__restrict__ X, int64_t xrs,
                                                               int64_t xcs, int64_t n,
                                                               const float *__restrict__ stats, bool norm_in,
                                                               float *__restrict__ Y, int64_t yrs, int64_t ycs) {
    // weights in matrix-operand order: layer l, block jb, K step kb, lane ->
    // W_l[16 jb + lane % 16][4 kb + lane / 16] (one conflict-free 256-byte
    // LDS read per operand); layer 3 padded to 32 rows with zeros; biases after
    constexpr int F1 = 0, F2 = F1 + MLP_H * MLP_IN, F3 = F2 + MLP_H * MLP_H, FB = F3 + 32 * MLP_H;
    __shared__ float W[FB + 2 * MLP_H + MLP_OUT];
    __shared__ float Hs[FWD_WAVES][FWD_MS * 16][FWD_HP];
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    for (int i = tid; i < FB; i += FWD_WAVES * 64) {
        int base, K, rows, ow;
        if (i < F2) { base = F1; K = MLP_IN; rows = MLP_H; ow = OW1; }
        else if (i < F3) { base = F2; K = MLP_H; rows = MLP_H; ow = OW2; }
        else { base = F3; K = MLP_H; rows = MLP_OUT; ow = OW3; }
        const int q = i - base, l = q & 63, kb = (q >> 6) % (K / 4), jb = (q >> 6) / (K / 4);
        const int row = 16 * jb + (l & 15), col = 4 * kb + (l >> 4);
        W[i] = row < rows ? wt<BF16W>(P, Pb, ow + row * K + col) : 0.0f;
    }
    for (int i = tid; i < 2 * MLP_H + MLP_OUT; i += FWD_WAVES * 64)
        W[FB + i] = wt<BF16W>(P, Pb, i < MLP_H ? OB1 + i : i < 2 * MLP_H ? OB2 + i - MLP_H : OB3 + i - 2 * MLP_H);
    __syncthreads();
    const int r16 = lane & 15, g = lane >> 4;
    // persistent over tiles of 256 samples: the weights are staged once per workgroup
    for (int64_t tile = blockIdx.x; tile * FWD_TILE < n; tile += gridDim.x) {
    const int64_t s0 = (tile * FWD_WAVES + w) * (FWD_MS * 16);
    float(*H)[FWD_HP] = Hs[w];
    f32x4 acc[4][FWD_MS];                          // [output block][sample block]
    auto zero = [&]() {
#pragma unroll
        for (int jb = 0; jb < 4; ++jb)
#pragma unroll
            for (int m = 0; m < FWD_MS; ++m) acc[jb][m] = f32x4{0, 0, 0, 0};
    };
    // layer 1: A straight from the inputs (standardised if asked; samples
    // past n are zero); all 120 values of the lane's operands are loaded
    // up front, so the tile waits for memory once
    zero();
    float xa[MLP_IN / 4][FWD_MS];
#pragma unroll
    for (int kb = 0; kb < MLP_IN / 4; ++kb)
#pragma unroll
        for (int m = 0; m < FWD_MS; ++m) {
            const int64_t sidx = s0 + 16 * m + r16;
            xa[kb][m] = sidx < n ? X[sidx * xrs + int64_t(4 * kb + g) * xcs] : 0.0f;
        }
#pragma unroll
    for (int kb = 0; kb < MLP_IN / 4; ++kb) {
        const int k = 4 * kb + g;
        float a[FWD_MS], b[4];
#pragma unroll
        for (int m = 0; m < FWD_MS; ++m) {
            a[m] = xa[kb][m];
            if (norm_in) a[m] = s0 + 16 * m + r16 < n ? (a[m] - stats[k]) / stats[MLP_IN + k] : 0.0f;
        }
#pragma unroll
        for (int jb = 0; jb < 4; ++jb) b[jb] = W[F1 + (jb * (MLP_IN / 4) + kb) * 64 + lane];
#pragma unroll
        for (int jb = 0; jb < 4; ++jb)
#pragma unroll
            for (int m = 0; m < FWD_MS; ++m) acc[jb][m] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[m], b[jb], acc[jb][m], 0, 0, 0);
    }
    auto to_h = [&](int ob) {
#pragma unroll
        for (int jb = 0; jb < 4; ++jb) {
            const int j = 16 * jb + r16;
            const float bias = W[FB + ob + j];
#pragma unroll
            for (int m = 0; m < FWD_MS; ++m)
#pragma unroll
                for (int r = 0; r < 4; ++r) H[16 * m + 4 * g + r][j] = fast_tanh(acc[jb][m][r] + bias);
        }
    };
    to_h(0);
    __syncthreads();
    // layer 2: A from the activations; the results stay in the accumulators
    // until every lane of the wavefront has read its operands, then replace them
    zero();
    for (int kb = 0; kb < MLP_H / 4; ++kb) {
        const int k = 4 * kb + g;
        float a[FWD_MS], b[4];
#pragma unroll
        for (int m = 0; m < FWD_MS; ++m) a[m] = H[16 * m + r16][k];
#pragma unroll
        for (int jb = 0; jb < 4; ++jb) b[jb] = W[F2 + (jb * (MLP_H / 4) + kb) * 64 + lane];
#pragma unroll
        for (int jb = 0; jb < 4; ++jb)
#pragma unroll
            for (int m = 0; m < FWD_MS; ++m) acc[jb][m] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[m], b[jb], acc[jb][m], 0, 0, 0);
    }
    __syncthreads();
    to_h(MLP_H);
    __syncthreads();
    // layer 3: 20 outputs in two blocks of 16 (the last 12 columns are zero
    // weights and are not stored)
    zero();
    for (int kb = 0; kb < MLP_H / 4; ++kb) {
        const int k = 4 * kb + g;
        float a[FWD_MS], b[2];
#pragma unroll
        for (int m = 0; m < FWD_MS; ++m) a[m] = H[16 * m + r16][k];
#pragma unroll
        for (int jb = 0; jb < 2; ++jb) b[jb] = W[F3 + (jb * (MLP_H / 4) + kb) * 64 + lane];
#pragma unroll
        for (int jb = 0; jb < 2; ++jb)
#pragma unroll
            for (int m = 0; m < FWD_MS; ++m) acc[jb][m] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[m], b[jb], acc[jb][m], 0, 0, 0);
    }
#pragma unroll
    for (int jb = 0; jb < 2; ++jb) {
        const int o = 16 * jb + r16;
        if (o >= MLP_OUT) continue;
        const float bias = W[FB + 2 * MLP_H + o];
        const float sc = stats ? stats[2 * MLP_IN + MLP_OUT + o] : 1.0f;
        const float mu = stats ? stats[2 * MLP_IN + o] : 0.0f;
#pragma unroll
        for (int m = 0; m < FWD_MS; ++m)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int64_t sidx = s0 + 16 * m + 4 * g + r;
                if (sidx < n) {
                    float z = acc[jb][m][r] + bias;
                    if (stats) z = z * sc + mu;
                    Y[sidx * yrs + int64_t(o) * ycs] = z;
                }
            }
    }
    __syncthreads();           // H is rewritten by the next tile
    }
}

// Gradient of L = sum_s |y_s - t_s|^2 / n over the samples idx[0..n) (or
// 0..n), FP32 master weights; with stats, rows are standardised on load
// (x - mu_x) / s_x and (t - mu_y) / s_y.
//
// A workgroup of eight wavefronts takes tiles of 32 samples, every product on
// the FP32 matrix cores: wavefront w owns the 16 x 16 output block (sample
// block w % 2, unit block w / 2) of each layer's forward and backward
// product, so the weight fragments it needs (83 registers) are loaded once
// and stay in registers over all its tiles, as do its seven blocks of the
// weight gradients (products of a tile's 32 samples as the K dimension).
// Activations and deltas pass through LDS with odd row strides.  A workgroup
// writes its row of partial gradients once, at the end (entry MLP_NPARAM is
// its loss); mlp_reduce_kernel adds the rows in order.  Bound by latency at
// the training loop's batch of 8,192 (256 tiles, one per CU: 0.5 GFLOP).
// One lane per sample with the weights from memory and 128 workgroups of one
// wavefront measured 866 us there, and its one-thread-per-parameter
// reduction 31 us; these two take 30 and 5.7 us.
constexpr int GRD_S = 32, GRD_THREADS = 512;
constexpr int GRD_XP = MLP_IN + 9, GRD_HP = MLP_H + 1, GRD_YP = 33;   // padded LDS rows (128 input columns are read)
__global__ __launch_bounds__(GRD_THREADS) void mlp_grad_kernel(const float *__restrict__ P,
                                                               const float *__restrict__ X,
                                                               const float *__restrict__ Tg,
                                                               const int32_t *__restrict__ idx,
                                                               int64_t n, const float *__restrict__ stats,
                                                               float *__restrict__ partial) {
    __shared__ float Xs[GRD_S][GRD_XP];
    __shared__ float H1[GRD_S][GRD_HP], H2[GRD_S][GRD_HP], D1[GRD_S][GRD_HP], D2[GRD_S][GRD_HP];
    __shared__ float St[MLP_NSTATS];                 // statistics (no statistics: 0 and 1, which change no value)
    __shared__ float DY[GRD_S][GRD_YP];              // targets, then 2 (y - t) / n; columns past the 20 outputs zero
    const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int r16 = lane & 15, g = lane >> 4;
    const int sb = 16 * (w & 1), jb = w >> 1;        // first sample, unit block of this wavefront
    const int unit = 16 * jb + r16;                  // the unit of this lane's accumulator column
    constexpr int K1 = MLP_IN / 4, K2 = MLP_H / 4, K3 = MLP_OUT / 4;

    // weight fragments: forward W_l[16 jb + lane % 16][4 kb + lane / 16],
    // backward (transposed products) W_l[4 kb + lane / 16][16 jb + lane % 16]
    // (all loads are issued before the first is waited for)
    float w1[K1], w2[K2], w3[K2], t3[K3], t2[K2];
    const int unit3 = min(unit, MLP_OUT - 1);        // rows past the outputs: a real row, zeroed below
#pragma unroll
    for (int kb = 0; kb < K1; ++kb) w1[kb] = P[OW1 + unit * MLP_IN + 4 * kb + g];
#pragma unroll
    for (int kb = 0; kb < K2; ++kb) {
        w2[kb] = P[OW2 + unit * MLP_H + 4 * kb + g];
        w3[kb] = P[OW3 + unit3 * MLP_H + 4 * kb + g];
        t2[kb] = P[OW2 + (4 * kb + g) * MLP_H + unit];
    }
#pragma unroll
    for (int kb = 0; kb < K3; ++kb) t3[kb] = P[OW3 + (4 * kb + g) * MLP_H + unit];
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int kb = 0; kb < K1; ++kb) w1[kb] = opaque(w1[kb]);
#pragma unroll
    for (int kb = 0; kb < K2; ++kb) {
        w2[kb] = opaque(w2[kb]);
        w3[kb] = opaque(unit < MLP_OUT ? w3[kb] : 0.0f);
        t2[kb] = opaque(t2[kb]);
    }
#pragma unroll
    for (int kb = 0; kb < K3; ++kb) t3[kb] = opaque(t3[kb]);
    const float bias1 = P[OB1 + unit], bias2 = P[OB2 + unit], bias3 = P[OB3 + unit3];

    for (int i = tid; i < MLP_NSTATS; i += GRD_THREADS)
        St[i] = stats ? stats[i] : (i < MLP_IN || (i >= 2 * MLP_IN && i < 2 * MLP_IN + MLP_OUT)) ? 0.0f : 1.0f;
    for (int i = tid; i < GRD_S * GRD_YP; i += GRD_THREADS) (&DY[0][0])[i] = 0.0f;
    for (int i = tid; i < GRD_S * GRD_XP; i += GRD_THREADS) (&Xs[0][0])[i] = 0.0f;

    f32x4 g1[4], g2[2], g3;                          // weight-gradient blocks
#pragma unroll
    for (int c = 0; c < 4; ++c) g1[c] = f32x4{0, 0, 0, 0};
    g2[0] = g2[1] = g3 = f32x4{0, 0, 0, 0};
    float gb = 0.0f, loss = 0.0f;                    // one bias gradient per thread (148 threads), the lane's losses

    const float inv_n = 1.0f / float(n);
    const int64_t ntiles = (n + GRD_S - 1) / GRD_S;
    // the tile's inputs and targets, fetched one tile ahead: 16 threads per
    // sample, input k = 16 q + tid % 16 (one row address per thread)
    const int fs = tid >> 4, fk = tid & 15;
    constexpr int NX = (MLP_IN + 15) / 16, NT = (MLP_OUT + 15) / 16;
    float xr[NX], tr[NT];
    auto fetch = [&](int64_t tile) {
        const int64_t s = tile * GRD_S + fs;
        const int64_t row = s < n ? (idx ? int64_t(idx[s]) : s) : 0;
        const float *x = X + row * MLP_IN + fk, *t = Tg + row * MLP_OUT + fk;
#pragma unroll
        for (int q = 0; q < NX; ++q) xr[q] = s < n && 16 * q + fk < MLP_IN ? x[16 * q] : 0.0f;
#pragma unroll
        for (int q = 0; q < NT; ++q) tr[q] = s < n && 16 * q + fk < MLP_OUT ? t[16 * q] : 0.0f;
    };
    // block of A[16 rows of LDS array a from sample sb][K] x fragments
    auto product = [&](const float *a, int stride, const float *frag, auto kc) {
        f32x4 acc{0, 0, 0, 0};
        constexpr int K = decltype(kc)::value;
#pragma unroll
        for (int kb = 0; kb < K; ++kb)
            acc = __builtin_amdgcn_mfma_f32_16x16x4f32(a[(sb + r16) * stride + 4 * kb + g], frag[kb], acc, 0, 0, 0);
        return acc;
    };
    fetch(blockIdx.x);
    for (int64_t tile = blockIdx.x; tile < ntiles; tile += gridDim.x) {
        __syncthreads();                             // the previous tile's arrays are free (and zeroed at first)
        const bool live = tile * GRD_S + fs < n;     // inputs of samples past n are zero
#pragma unroll
        for (int q = 0; q < NX; ++q) {
            const int k = 16 * q + fk;
            if (k < MLP_IN) Xs[fs][k] = live ? (xr[q] - St[k]) / St[MLP_IN + k] : 0.0f;
        }
#pragma unroll
        for (int q = 0; q < NT; ++q) {
            const int o = 16 * q + fk;
            if (o < MLP_OUT) DY[fs][o] = (tr[q] - St[2 * MLP_IN + o]) / St[2 * MLP_IN + MLP_OUT + o];
        }
        __syncthreads();
        if (tile + gridDim.x < ntiles) fetch(tile + gridDim.x);
        const f32x4 z1 = product(&Xs[0][0], GRD_XP, w1, std::integral_constant<int, K1>{});
        float h1[4], h2[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) H1[sb + 4 * g + r][unit] = h1[r] = tanhf(z1[r] + bias1);
        __syncthreads();
        const f32x4 z2 = product(&H1[0][0], GRD_HP, w2, std::integral_constant<int, K2>{});
#pragma unroll
        for (int r = 0; r < 4; ++r) H2[sb + 4 * g + r][unit] = h2[r] = tanhf(z2[r] + bias2);
        __syncthreads();
        if (jb < 2) {
            const f32x4 y = product(&H2[0][0], GRD_HP, w3, std::integral_constant<int, K2>{});
            if (unit < MLP_OUT) {
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const int s = sb + 4 * g + r;
                    const float d = tile * GRD_S + s < n ? y[r] + bias3 - DY[s][unit] : 0.0f;
                    loss += d * d;
                    DY[s][unit] = 2.0f * d * inv_n;
                }
            }
        }
        __syncthreads();
        // dz2 = (W3^T dy) (1 - h2^2), dz1 = (W2^T dz2) (1 - h1^2)
        const f32x4 e2 = product(&DY[0][0], GRD_YP, t3, std::integral_constant<int, K3>{});
#pragma unroll
        for (int r = 0; r < 4; ++r) D2[sb + 4 * g + r][unit] = e2[r] * (1.0f - h2[r] * h2[r]);
        __syncthreads();
        const f32x4 e1 = product(&D2[0][0], GRD_HP, t2, std::integral_constant<int, K2>{});
#pragma unroll
        for (int r = 0; r < 4; ++r) D1[sb + 4 * g + r][unit] = e1[r] * (1.0f - h1[r] * h1[r]);
        // weight gradients: row block jb of dW2 and dW1, two and four column
        // blocks; block (w % 2, w / 2) of dW3
#pragma unroll
        for (int kb = 0; kb < GRD_S / 4; ++kb) {
            const int s = 4 * kb + g;
            const float a2 = D2[s][unit], a3 = DY[s][16 * (w & 1) + r16];
            g3 = __builtin_amdgcn_mfma_f32_16x16x4f32(a3, H2[s][unit], g3, 0, 0, 0);
#pragma unroll
            for (int c = 0; c < 2; ++c)
                g2[c] = __builtin_amdgcn_mfma_f32_16x16x4f32(a2, H1[s][16 * (2 * (w & 1) + c) + r16], g2[c], 0, 0, 0);
        }
        __syncthreads();
#pragma unroll
        for (int kb = 0; kb < GRD_S / 4; ++kb) {
            const int s = 4 * kb + g;
            const float a1 = D1[s][unit];
#pragma unroll
            for (int c = 0; c < 4; ++c)
                g1[c] = __builtin_amdgcn_mfma_f32_16x16x4f32(a1, Xs[s][16 * (4 * (w & 1) + c) + r16], g1[c], 0, 0, 0);
        }
        if (tid < 2 * MLP_H + MLP_OUT)
            for (int s = 0; s < GRD_S; ++s)
                gb += tid < MLP_H ? D1[s][tid] : tid < 2 * MLP_H ? D2[s][tid - MLP_H] : DY[s][tid - 2 * MLP_H];
    }
    float *part = partial + int64_t(blockIdx.x) * (MLP_NPARAM + 1);
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const int row = 16 * jb + 4 * g + r;
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            const int k = 16 * (4 * (w & 1) + c) + r16;
            if (k < MLP_IN) part[OW1 + row * MLP_IN + k] = g1[c][r];
        }
#pragma unroll
        for (int c = 0; c < 2; ++c) part[OW2 + row * MLP_H + 16 * (2 * (w & 1) + c) + r16] = g2[c][r];
        const int o = 16 * (w & 1) + 4 * g + r;
        if (o < MLP_OUT) part[OW3 + o * MLP_H + unit] = g3[r];
    }
    if (tid < 2 * MLP_H + MLP_OUT)
        part[tid < MLP_H ? OB1 + tid : tid < 2 * MLP_H ? OB2 + tid - MLP_H : OB3 + tid - 2 * MLP_H] = gb;
    // the workgroup's loss: lanes in a fixed tree, then the four wavefronts
    // that hold outputs in order
    for (int o = 32; o; o >>= 1) loss += __shfl_down(loss, o);
    __syncthreads();
    if (lane == 0) H1[0][w] = loss;
    __syncthreads();
    if (tid == 0) part[MLP_NPARAM] = (((H1[0][0] + H1[0][1]) + H1[0][2]) + H1[0][3]) * inv_n;
}

// grad[p] = sum over blocks of partial[b][p]: 64 parameters per workgroup,
// each of its 16 wavefronts sums a run of blocks in order and the runs are
// added in order (deterministic)
constexpr int RDC_WAVES = 16;
__global__ __launch_bounds__(64 * RDC_WAVES) void mlp_reduce_kernel(const float *__restrict__ partial,
                                                                    int nblk, float *__restrict__ grad) {
    __shared__ float sh[RDC_WAVES][64];
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, p = blockIdx.x * 64 + lane;
    const int run = (nblk + RDC_WAVES - 1) / RDC_WAVES, b1 = min(nblk, (w + 1) * run);
    float s = 0.0f;
    if (p <= MLP_NPARAM)
#pragma unroll 8
        for (int b = w * run; b < b1; ++b) s += partial[int64_t(b) * (MLP_NPARAM + 1) + p];
    sh[w][lane] = s;
    __syncthreads();
    if (w || p > MLP_NPARAM) return;
    s = sh[0][lane];
    for (int q = 1; q < RDC_WAVES; ++q) s += sh[q][lane];
    grad[p] = s;
}

// Adam (Kingma & Ba): m = b1 m + (1-b1) g, v = b2 v + (1-b2) g^2,
// p -= lr (m / c1) / (sqrt(v / c2) + eps); also refresh the BF16 copy.
__global__ __launch_bounds__(256) void adam_kernel(float *__restrict__ P, const float *__restrict__ G,
                                                   float *__restrict__ M, float *__restrict__ V,
                                                   float lr, float b1, float b2, float eps, float c1,
                                                   float c2, uint16_t *__restrict__ Pb) {
    const int p = blockIdx.x * blockDim.x + threadIdx.x;
    if (p >= MLP_NPARAM) return;
    const float g = G[p];
    const float m = b1 * M[p] + (1.0f - b1) * g;
    const float v = b2 * V[p] + (1.0f - b2) * g * g;
    M[p] = m;
    V[p] = v;
    const float w = P[p] - lr * (m / c1) / (sqrtf(v / c2) + eps);
    P[p] = w;
    uint32_t b = __builtin_bit_cast(uint32_t, w);
    b += 0x7fffu + ((b >> 16) & 1u);   // round to nearest even
    Pb[p] = uint16_t(b >> 16);
}

__global__ __launch_bounds__(256) void to_bf16_kernel(const float *__restrict__ P, uint16_t *__restrict__ Pb) {
    const int p = blockIdx.x * blockDim.x + threadIdx.x;
    if (p >= MLP_NPARAM) return;
    uint32_t b = __builtin_bit_cast(uint32_t, P[p]);
    b += 0x7fffu + ((b >> 16) & 1u);
    Pb[p] = uint16_t(b >> 16);
}

}  // namespace

template <typename T>
hipError_t launch_moments(const T *U, const T *B, int64_t ld, int64_t nelem, int nu, const float *Mom,
                          float *mom, int64_t goff, int64_t rs, int64_t cs, const float *ystats,
                          hipStream_t s) {
    if (!nelem) return hipSuccess;
    moments_kernel<T><<<unsigned((nelem + 255) / 256), 256, 0, s>>>(U, B, ld, nelem, nu, Mom, mom, goff, rs,
                                                                    cs, ystats);
    return hipGetLastError();
}

hipError_t launch_features(const float *mom, int64_t rs, int64_t cs, const int32_t *nb, int64_t ntot,
                           const float *stats, float *feat, int64_t frs, int64_t fcs, hipStream_t s) {
    if (!ntot) return hipSuccess;
    features_kernel<<<dim3(unsigned((ntot + 255) / 256), 6), 256, 0, s>>>(mom, rs, cs, nb, ntot, stats, feat, frs, fcs);
    return hipGetLastError();
}

hipError_t launch_mlp_forward(const float *P, const uint16_t *Pb, bool bf16, const float *X, int64_t xrs,
                              int64_t xcs, int64_t n, const float *stats, bool norm_in, float *Y, int64_t yrs,
                              int64_t ycs, hipStream_t s) {
    if (!n) return hipSuccess;
    // one workgroup per CU (the staged weights and activations take 119 KB
    // of LDS), each looping over tiles of FWD_TILE samples
    const int64_t tiles = (n + FWD_TILE - 1) / FWD_TILE;
    const unsigned g = unsigned(tiles < 256 ? tiles : 256);
    norm_in = norm_in && stats;
    if (bf16)
        mlp_forward_mfma_kernel<true><<<g, FWD_WAVES * 64, 0, s>>>(P, Pb, X, xrs, xcs, n, stats, norm_in, Y, yrs, ycs);
    else
        mlp_forward_mfma_kernel<false><<<g, FWD_WAVES * 64, 0, s>>>(P, Pb, X, xrs, xcs, n, stats, norm_in, Y, yrs,
                                                                   ycs);
    return hipGetLastError();
}

hipError_t launch_mlp_grad(const float *P, const float *X, const float *Tg, const int32_t *idx, int64_t n,
                           const float *stats, float *partial, int nblk, float *grad, hipStream_t s) {
    if (n <= 0) return hipErrorInvalidValue;
    const int64_t tiles = (n + GRD_S - 1) / GRD_S;
    const int g = int(tiles < nblk ? tiles : nblk);
    mlp_grad_kernel<<<g, GRD_THREADS, 0, s>>>(P, X, Tg, idx, n, stats, partial);
    mlp_reduce_kernel<<<(MLP_NPARAM + 1 + 63) / 64, 64 * RDC_WAVES, 0, s>>>(partial, g, grad);
    return hipGetLastError();
}

hipError_t launch_adam(float *P, const float *G, float *M, float *V, float lr, float b1, float b2, float eps,
                       int t, uint16_t *Pb, hipStream_t s) {
    const float c1 = 1.0f - powf(b1, float(t)), c2 = 1.0f - powf(b2, float(t));
    adam_kernel<<<(MLP_NPARAM + 255) / 256, 256, 0, s>>>(P, G, M, V, lr, b1, b2, eps, c1, c2, Pb);
    return hipGetLastError();
}

hipError_t launch_to_bf16(const float *P, uint16_t *Pb, hipStream_t s) {
    to_bf16_kernel<<<(MLP_NPARAM + 255) / 256, 256, 0, s>>>(P, Pb);
    return hipGetLastError();
}

template hipError_t launch_moments<float>(const float *, const float *, int64_t, int64_t, int, const float *,
                                          float *, int64_t, int64_t, int64_t, const float *, hipStream_t);
template hipError_t launch_moments<double>(const double *, const double *, int64_t, int64_t, int,
                                           const float *, float *, int64_t, int64_t, int64_t, const float *,
                                           hipStream_t);

}  // namespace frd
