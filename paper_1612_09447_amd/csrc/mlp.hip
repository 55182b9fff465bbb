// Start-vector network for the learned form: a multilayer perceptron
// 32 -> 64 -> 64 -> 16 (SiLU hidden activations, linear output) trained online
// with mean-squared error and Adam. Sec. IV of the paper builds CG start
// vectors from a POD basis of earlier solutions; here the small reduced solve
// is replaced by this learned map, and CG stays the judge of the result.
//
// One workgroup runs a whole minibatch (B <= 64): forward, loss, backward and
// the Adam update, all in one launch with the matmul weights and the
// activations in LDS; a forward pass alone takes one workgroup per 64 rows.
// Matmul operands are rounded to bfloat16 (round to nearest even) in BF16
// mode, products accumulate in FP32; master weights, gradients and Adam
// moments are FP32. Every sum runs in a fixed order, so results are
// deterministic.
#include <hip/hip_runtime.h>

#include <cmath>
#include <cstdint>
#include <cstring>
#include <string>
#include <vector>

#include "eqs_internal.h"

namespace eqs {

constexpr int kIn = 32, kH = 64, kOut = 16, kMaxB = 64;
constexpr int oW1 = 0, oB1 = oW1 + kH * kIn, oW2 = oB1 + kH, oB2 = oW2 + kH * kH, oW3 = oB2 + kH,
              oB3 = oW3 + kOut * kH, kNParam = oB3 + kOut;
static_assert(kNParam == 7312, "parameter layout");

__device__ __forceinline__ float bf16_round(float x) {
    uint32_t u = __float_as_uint(x);
    if ((u & 0x7f800000u) == 0x7f800000u) return x;  // inf / nan unchanged
    u = (u + 0x7fffu + ((u >> 16) & 1u)) & 0xffff0000u;
    return __uint_as_float(u);
}

template <bool BF16>
__device__ __forceinline__ float q(float x) {
    return BF16 ? bf16_round(x) : x;
}

__device__ __forceinline__ float silu(float z) { return z / (1.0f + expf(-z)); }
__device__ __forceinline__ float silu_grad(float z) {
    const float s = 1.0f / (1.0f + expf(-z));
    return s * (1.0f + z * (1.0f - s));
}

struct MlpState {
    float lr, beta1, beta2, eps;
    int32_t step;  // Adam steps taken
    float loss;    // loss of the last training batch
};

// ---- tiles of the minibatch products -------------------------------------
// One workgroup of kThreads threads; rows of every LDS array are padded by 4
// floats (row strides 36, 68, 20: 16-byte rows whose starts spread over the
// banks). A thread owns a TI x TJ tile of a product's output, held in
// registers: per four terms of the sum it reads TI + TJ 16-byte pieces for
// 4 TI TJ multiply-adds (the untiled form read two words for each one).
// Every sum runs over k (or over the batch) in increasing order with one
// accumulator per output.
constexpr int kThreads = 512;
constexpr int sK1 = kIn + 4, sK2 = kH + 4, sK3 = kOut + 4;  // row strides (floats)

// C[i][j] = sum_k A[i][k] B[j][k], k = 0..K-1 contiguous in both; the thread's
// rows are i0 + SI u, its columns j0 + SJ v (strided, so that the lanes of a
// read instruction take neighbouring rows, which sit in different banks).
template <int TI, int TJ, int SI, int SJ, int K, int SA, int SB>
__device__ __forceinline__ void tile_dot(const float* __restrict__ A, const float* __restrict__ B, int i0, int j0,
                                         float (&c)[TI][TJ]) {
#pragma unroll
    for (int u = 0; u < TI; ++u)
#pragma unroll
        for (int v = 0; v < TJ; ++v) c[u][v] = 0.0f;
#pragma unroll 4
    for (int k = 0; k < K; k += 4) {
        float4 a[TI], b[TJ];
#pragma unroll
        for (int u = 0; u < TI; ++u) a[u] = *reinterpret_cast<const float4*>(A + (i0 + SI * u) * SA + k);
#pragma unroll
        for (int v = 0; v < TJ; ++v) b[v] = *reinterpret_cast<const float4*>(B + (j0 + SJ * v) * SB + k);
#pragma unroll
        for (int u = 0; u < TI; ++u)
#pragma unroll
            for (int v = 0; v < TJ; ++v) {
                c[u][v] += b[v].x * a[u].x;
                c[u][v] += b[v].y * a[u].y;
                c[u][v] += b[v].z * a[u].z;
                c[u][v] += b[v].w * a[u].w;
            }
    }
}

template <int N>
__device__ __forceinline__ void load_row(const float* __restrict__ p, float (&r)[N]) {
    if constexpr (N == 4) {
        const float4 v = *reinterpret_cast<const float4*>(p);
        r[0] = v.x; r[1] = v.y; r[2] = v.z; r[3] = v.w;
    } else if constexpr (N == 2) {
        const float2 v = *reinterpret_cast<const float2*>(p);
        r[0] = v.x; r[1] = v.y;
    } else {
        r[0] = p[0];
    }
}

// C[i0 + u][j0 + v] = sum_n A[n][i0 + u] B[n][j0 + v], n = 0..n_rows-1.
template <int TI, int TJ, int SA, int SB>
__device__ __forceinline__ void tile_outer(const float* __restrict__ A, const float* __restrict__ B, int n_rows,
                                           int i0, int j0, float (&c)[TI][TJ]) {
#pragma unroll
    for (int u = 0; u < TI; ++u)
#pragma unroll
        for (int v = 0; v < TJ; ++v) c[u][v] = 0.0f;
#pragma unroll 4
    for (int n = 0; n < n_rows; ++n) {
        float a[TI], b[TJ];
        load_row<TI>(A + n * SA + i0, a);
        load_row<TJ>(B + n * SB + j0, b);
#pragma unroll
        for (int u = 0; u < TI; ++u)
#pragma unroll
            for (int v = 0; v < TJ; ++v) c[u][v] += a[u] * b[v];
    }
}

// C[i0 + SI u][j0 + v] = sum_o A[i0 + SI u][o] W[o][j0 + v], o = 0..K-1.
template <int TI, int TJ, int SI, int K, int SA, int SW>
__device__ __forceinline__ void tile_back(const float* __restrict__ A, const float* __restrict__ W, int i0, int j0,
                                          float (&c)[TI][TJ]) {
#pragma unroll
    for (int u = 0; u < TI; ++u)
#pragma unroll
        for (int v = 0; v < TJ; ++v) c[u][v] = 0.0f;
#pragma unroll 2
    for (int o = 0; o < K; o += 4) {
        float a[TI][4], w[4][TJ];
#pragma unroll
        for (int u = 0; u < TI; ++u) load_row<4>(A + (i0 + SI * u) * SA + o, a[u]);
#pragma unroll
        for (int d = 0; d < 4; ++d) load_row<TJ>(W + (o + d) * SW + j0, w[d]);
#pragma unroll
        for (int d = 0; d < 4; ++d)
#pragma unroll
            for (int u = 0; u < TI; ++u)
#pragma unroll
                for (int v = 0; v < TJ; ++v) c[u][v] += a[u][d] * w[d][v];
    }
}

// Adam (Kingma & Ba) on one parameter; m1, m2 and master were read at entry.
struct Moments {
    float w, a, v;
};
struct AdamConst {
    float lr, beta1, beta2, eps, bc1, bc2;
};
template <bool BF16>
__device__ __forceinline__ void adam(const AdamConst& A, const Moments& o, int i, float g, float* __restrict__ master,
                                     float* __restrict__ wq, float* __restrict__ grad, float* __restrict__ m1,
                                     float* __restrict__ m2) {
    grad[i] = g;
    const float a = A.beta1 * o.a + (1.0f - A.beta1) * g;
    const float v = A.beta2 * o.v + (1.0f - A.beta2) * g * g;
    m1[i] = a;
    m2[i] = v;
    const float w = o.w - A.lr * (a / A.bc1) / (sqrtf(v / A.bc2) + A.eps);
    master[i] = w;
    wq[i] = q<BF16>(w);
}

// wq: matmul copies of the weights (bf16-rounded in BF16 mode); master: FP32.
// Forward (grid: one workgroup per kMaxB rows of x) or one training step (one
// workgroup, B <= kMaxB): everything between the reads of the weights and the
// writes of the results stays in LDS (137 KiB of gfx950's 160 KiB when
// training) and registers. Operands of the products are rounded once, when
// they are written; the parameters' Adam state is read at entry, so its
// latency passes behind the forward products. One workgroup is bound by the
// LDS reads and multiply-adds of its own CU: the 1.25 M multiply-adds of a
// 64-row step take 8 us at 64 per clock and 2.4 GHz.
// (Matrix instructions would shorten those 8 us, at another order of the sums;
// the phases' barriers and the Adam state's traffic would stay.)
template <bool TRAIN, bool BF16>
__global__ __launch_bounds__(kThreads) void k_mlp(const float* __restrict__ x, const float* __restrict__ tgt,
                                                  float* __restrict__ y, int32_t B, float* __restrict__ master,
                                                  float* __restrict__ wq, float* __restrict__ grad,
                                                  float* __restrict__ m1, float* __restrict__ m2,
                                                  MlpState* __restrict__ st) {
    __shared__ __align__(16) float sw1[kH * sK1], sw2[kH * sK2], sw3[kOut * sK2];  // matmul weights
    __shared__ float sb[kH + kH + kOut];                                            // biases (master)
    __shared__ __align__(16) float sx[kMaxB * sK1];
    __shared__ __align__(16) float sa1[kMaxB * sK2], sa2[kMaxB * sK2];  // activations as operands
    __shared__ __align__(16) float sh1[TRAIN ? kMaxB * sK2 : 4], sh2[TRAIN ? kMaxB * sK2 : 4];
    __shared__ __align__(16) float sd2[TRAIN ? kMaxB * sK2 : 4];                    // dh2 as an operand
    __shared__ __align__(16) float sy[kMaxB * sK3], syq[TRAIN ? kMaxB * sK3 : 4];  // y, then dy (and as an operand)
    __shared__ float sred[kThreads / 64];
    const int tid = threadIdx.x;
    if (!TRAIN) {  // this workgroup's rows
        const int32_t b0 = (int32_t)blockIdx.x * kMaxB;
        x += (int64_t)b0 * kIn;
        y += (int64_t)b0 * kOut;
        B = min(B - b0, kMaxB);
    }

    for (int i = tid; i < kH * kIn / 4; i += kThreads)
        *reinterpret_cast<float4*>(sw1 + (i / (kIn / 4)) * sK1 + 4 * (i % (kIn / 4))) =
            reinterpret_cast<const float4*>(wq + oW1)[i];
    for (int i = tid; i < kH * kH / 4; i += kThreads)
        *reinterpret_cast<float4*>(sw2 + (i / (kH / 4)) * sK2 + 4 * (i % (kH / 4))) =
            reinterpret_cast<const float4*>(wq + oW2)[i];
    for (int i = tid; i < kOut * kH / 4; i += kThreads)
        *reinterpret_cast<float4*>(sw3 + (i / (kH / 4)) * sK2 + 4 * (i % (kH / 4))) =
            reinterpret_cast<const float4*>(wq + oW3)[i];
    if (tid < kH) sb[tid] = master[oB1 + tid];
    else if (tid < 2 * kH) sb[tid] = master[oB2 + tid - kH];
    else if (tid < 2 * kH + kOut) sb[tid] = master[oB3 + tid - 2 * kH];
    for (int i = tid; i < kMaxB * kIn; i += kThreads)  // rows past B are zero
        sx[(i / kIn) * sK1 + i % kIn] = i < B * kIn ? q<BF16>(x[i]) : 0.0f;

    // The tiles of this thread: 64 x 64 outputs as 2 x 4, 64 x 32 as 2 x 2, 64 x 16 as 2 x 1.
    const int tr = tid >> 4, tc = tid & 15;  // 32 x 16 threads
    AdamConst ac{};
    Moments p1[2][2], p2[2][4], p3[2], pb{};  // W1 (o = 2 tr + u, k = 2 tc + v), W2 (2 tr + u, 4 tc + v), W3, bias
    if (TRAIN) {
        auto rd = [&](int i) { return Moments{master[i], m1[i], m2[i]}; };
#pragma unroll
        for (int u = 0; u < 2; ++u) {
#pragma unroll
            for (int v = 0; v < 2; ++v) p1[u][v] = rd(oW1 + (2 * tr + u) * kIn + 2 * tc + v);
#pragma unroll
            for (int v = 0; v < 4; ++v) p2[u][v] = rd(oW2 + (2 * tr + u) * kH + 4 * tc + v);
        }
        // W3 (16 x 64): thread -> row tid / 32, columns 2 (tid % 32) + v
#pragma unroll
        for (int v = 0; v < 2; ++v) p3[v] = rd(oW3 + (tid >> 5) * kH + 2 * (tid & 31) + v);
        const int ib = tid < kH ? oB1 + tid : tid < 2 * kH ? oB2 + tid - kH : oB3 + min(tid - 2 * kH, kOut - 1);
        pb = rd(ib);
        const int t = st->step + 1;
        ac = AdamConst{st->lr, st->beta1, st->beta2, st->eps, 1.0f - powf(st->beta1, (float)t),
                       1.0f - powf(st->beta2, (float)t)};
    }
    __syncthreads();
    // h1 = W1 x + b1, a1 = silu(h1): rows tr + 32 u, columns tc + 16 v
    {
        float c[2][4];
        tile_dot<2, 4, 32, 16, kIn, sK1, sK1>(sx, sw1, tr, tc, c);
#pragma unroll
        for (int u = 0; u < 2; ++u)
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int b = tr + 32 * u, o = tc + 16 * v;
                const float h = c[u][v] + sb[o];
                if (TRAIN) sh1[b * sK2 + o] = h;
                sa1[b * sK2 + o] = q<BF16>(silu(h));
            }
    }
    __syncthreads();
    // h2 = W2 a1 + b2, a2 = silu(h2)
    {
        float c[2][4];
        tile_dot<2, 4, 32, 16, kH, sK2, sK2>(sa1, sw2, tr, tc, c);
#pragma unroll
        for (int u = 0; u < 2; ++u)
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int b = tr + 32 * u, o = tc + 16 * v;
                const float h = c[u][v] + sb[kH + o];
                if (TRAIN) sh2[b * sK2 + o] = h;
                sa2[b * sK2 + o] = q<BF16>(silu(h));
            }
    }
    __syncthreads();
    // y = W3 a2 + b3; with the targets also dy = 2 (y - t) / (16 B) and the loss
    {
        float c[2][1];
        tile_dot<2, 1, 32, 16, kH, sK2, sK2>(sa2, sw3, tr, tc, c);
        float part = 0.0f;
        const float inv = 1.0f / (float)(B * kOut);
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            const int b = tr + 32 * u;
            const float v = c[u][0] + sb[2 * kH + tc];
            if (!TRAIN) {
                if (b < B) y[b * kOut + tc] = v;
            } else {
                float dy = 0.0f;
                if (b < B) {
                    const float d = v - tgt[b * kOut + tc];
                    part += d * d;
                    dy = 2.0f * d * inv;
                }
                sy[b * sK3 + tc] = dy;
                syq[b * sK3 + tc] = q<BF16>(dy);
            }
        }
        if (!TRAIN) return;
        for (int off = 32; off > 0; off >>= 1) part += __shfl_down(part, off, 64);
        if ((tid & 63) == 0) sred[tid >> 6] = part;
    }
    __syncthreads();
    // dh2 = (dy W3) silu'(h2): sh2 keeps it, sd2 holds it as an operand
    {
        float c[2][4];
        tile_back<2, 4, 32, kOut, sK3, sK2>(syq, sw3, tr, 4 * tc, c);
#pragma unroll
        for (int u = 0; u < 2; ++u)
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int at = (tr + 32 * u) * sK2 + 4 * tc + v;
                const float d = c[u][v] * silu_grad(sh2[at]);
                sh2[at] = d;
                sd2[at] = q<BF16>(d);
            }
    }
    // layer 3: gW3 = dy^T a2, gb3 = sum_b dy
    {
        float c[1][2];
        const int o = tid >> 5, k = 2 * (tid & 31);
        tile_outer<1, 2, sK3, sK2>(syq, sa2, B, o, k, c);
#pragma unroll
        for (int v = 0; v < 2; ++v) adam<BF16>(ac, p3[v], oW3 + o * kH + k + v, c[0][v], master, wq, grad, m1, m2);
    }
    if (tid == 0) {
        float s = 0.0f;
        for (int k = 0; k < kThreads / 64; ++k) s += sred[k];
        st->loss = s * (1.0f / (float)(B * kOut));
    }
    __syncthreads();
    // dh1 = (dh2 W2) silu'(h1) over sh1, and over sa2 (free now) as an operand
    {
        float c[2][4];
        tile_back<2, 4, 32, kH, sK2, sK2>(sd2, sw2, tr, 4 * tc, c);
#pragma unroll
        for (int u = 0; u < 2; ++u)
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int at = (tr + 32 * u) * sK2 + 4 * tc + v;
                const float d = c[u][v] * silu_grad(sh1[at]);
                sh1[at] = d;
                sa2[at] = q<BF16>(d);
            }
    }
    // layer 2: gW2 = dh2^T a1
    {
        float c[2][4];
        tile_outer<2, 4, sK2, sK2>(sd2, sa1, B, 2 * tr, 4 * tc, c);
#pragma unroll
        for (int u = 0; u < 2; ++u)
#pragma unroll
            for (int v = 0; v < 4; ++v)
                adam<BF16>(ac, p2[u][v], oW2 + (2 * tr + u) * kH + 4 * tc + v, c[u][v], master, wq, grad, m1, m2);
    }
    __syncthreads();
    // layer 1: gW1 = dh1^T x
    {
        float c[2][2];
        tile_outer<2, 2, sK2, sK1>(sa2, sx, B, 2 * tr, 2 * tc, c);
#pragma unroll
        for (int u = 0; u < 2; ++u)
#pragma unroll
            for (int v = 0; v < 2; ++v)
                adam<BF16>(ac, p1[u][v], oW1 + (2 * tr + u) * kIn + 2 * tc + v, c[u][v], master, wq, grad, m1, m2);
    }
    // biases: column sums of dh1, dh2 and dy
    if (tid < 2 * kH + kOut) {
        const float* col = tid < kH ? sh1 + tid : tid < 2 * kH ? sh2 + tid - kH : sy + tid - 2 * kH;
        const int ld = tid < 2 * kH ? sK2 : sK3;
        float acc = 0.0f;
#pragma unroll 8
        for (int b = 0; b < B; ++b) acc += col[b * ld];
        const int ib = tid < kH ? oB1 + tid : tid < 2 * kH ? oB2 + tid - kH : oB3 + tid - 2 * kH;
        adam<BF16>(ac, pb, ib, acc, master, wq, grad, m1, m2);
    }
    if (tid == 0) st->step += 1;
}

// Inference for one feature vector, followed by the map from the network's
// 16 outputs to the 16 snapshot coefficients of the start vector:
// alpha = bias + P y (P carries the POD basis change and the output scale).
// With a guard block g (K = V^T M V [16 x 16], d = V^T (r_j - r_{j-1}) [16],
// scale s) the correction c = s y is kept only if it lowers the M-norm of the
// error of the start vector: |x* - x0 - V c|_M^2 = |x* - x0|_M^2 - (2 c.d -
// c.K c) when M x0 = r_{j-1}, so the test needs no product with M; otherwise
// alpha = bias. stat[0] / stat[1] count kept / dropped corrections.
struct MlpIn {
    float x[kIn];
    double P[kOut * kOut];
    double bias[kOut];
};

template <int K>
__device__ __forceinline__ void alpha_row(const float* __restrict__ w, float4 (&r)[K / 4]) {
#pragma unroll
    for (int k = 0; k < K / 4; ++k) r[k] = reinterpret_cast<const float4*>(w)[k];
}
template <int K>
__device__ __forceinline__ float alpha_dot(const float4 (&r)[K / 4], const float* __restrict__ a) {
    float acc = 0.0f;
#pragma unroll
    for (int k = 0; k < K / 4; ++k) {
        acc += r[k].x * a[4 * k];
        acc += r[k].y * a[4 * k + 1];
        acc += r[k].z * a[4 * k + 2];
        acc += r[k].w * a[4 * k + 3];
    }
    return acc;
}

// Every weight row and guard row of a thread is read at entry with 16-byte
// loads, so the launch waits for memory once, not once per layer and per term.
template <bool BF16>
__global__ __launch_bounds__(64) void k_mlp_alpha(MlpIn in, const float* __restrict__ master,
                                                   const float* __restrict__ wq, double* __restrict__ alpha,
                                                   const double* __restrict__ guard, int32_t* __restrict__ stat) {
    __shared__ float xq[kIn], a1[kH], a2[kH], yv[kOut];
    __shared__ double gy[2 * kOut];  // yv[p] d[p], then yv[p] (K yv)[p]
    __shared__ int take;
    const int tid = threadIdx.x, o3 = tid & (kOut - 1);
    float4 w1[kIn / 4], w2[kH / 4], w3[kH / 4];
    alpha_row<kIn>(wq + oW1 + tid * kIn, w1);
    alpha_row<kH>(wq + oW2 + tid * kH, w2);
    alpha_row<kH>(wq + oW3 + o3 * kH, w3);
    const float b1 = master[oB1 + tid], b2 = master[oB2 + tid], b3 = master[oB3 + o3];
    double grow[kOut], gd = 0.0, gs = 0.0;
    if (guard) {
#pragma unroll
        for (int k = 0; k < kOut; ++k) grow[k] = guard[o3 * kOut + k];
        gd = guard[kOut * kOut + o3];
        gs = guard[kOut * kOut + kOut];
    }
    if (tid < kIn) xq[tid] = q<BF16>(in.x[tid]);
    __syncthreads();
    a1[tid] = q<BF16>(silu(alpha_dot<kIn>(w1, xq) + b1));
    __syncthreads();
    a2[tid] = q<BF16>(silu(alpha_dot<kH>(w2, a1) + b2));
    __syncthreads();
    if (tid < kOut) yv[tid] = alpha_dot<kH>(w3, a2) + b3;
    __syncthreads();
    if (guard && tid < kOut) {
        double ky = 0.0;
#pragma unroll
        for (int k = 0; k < kOut; ++k) ky += grow[k] * (double)yv[k];
        gy[tid] = (double)yv[tid] * gd;
        gy[kOut + tid] = (double)yv[tid] * ky;
    }
    __syncthreads();
    if (tid == 0) {
        take = 1;
        if (guard) {
            double yd = 0.0, yky = 0.0;
            for (int p = 0; p < kOut; ++p) {
                yd += gy[p];
                yky += gy[kOut + p];
            }
            const double gain = 2.0 * gs * yd - gs * gs * yky;
            take = gain > 0.0 ? 1 : 0;
            stat[take ? 0 : 1] += 1;
        }
    }
    __syncthreads();
    if (tid < kOut) {
        double acc = in.bias[tid];
        if (take)
            for (int k = 0; k < kOut; ++k) acc += in.P[tid * kOut + k] * (double)yv[k];
        alpha[tid] = acc;
    }
}

}  // namespace eqs

struct eqs_mlp {
    int device = 0;
    hipStream_t stream = nullptr;
    eqs_ctx* owner = nullptr;  // context whose device memory holds the buffers, or NULL
    int bf16 = 1;
    float *master = nullptr, *wq = nullptr, *grad = nullptr, *m1 = nullptr, *m2 = nullptr;
    eqs::MlpState* st = nullptr;
};

namespace eqs {

static void mlp_launch(eqs_mlp* n, bool train, const float* x, const float* t, float* y, int32_t B) {
    const dim3 g(train ? 1u : (unsigned)((B + kMaxB - 1) / kMaxB)), b(kThreads);
    if (train) {
        if (n->bf16)
            hipLaunchKernelGGL((k_mlp<true, true>), g, b, 0, n->stream, x, t, y, B, n->master, n->wq, n->grad, n->m1,
                               n->m2, n->st);
        else
            hipLaunchKernelGGL((k_mlp<true, false>), g, b, 0, n->stream, x, t, y, B, n->master, n->wq, n->grad, n->m1,
                               n->m2, n->st);
    } else {
        if (n->bf16)
            hipLaunchKernelGGL((k_mlp<false, true>), g, b, 0, n->stream, x, t, y, B, n->master, n->wq, n->grad,
                               n->m1, n->m2, n->st);
        else
            hipLaunchKernelGGL((k_mlp<false, false>), g, b, 0, n->stream, x, t, y, B, n->master, n->wq, n->grad,
                               n->m1, n->m2, n->st);
    }
}

static float host_bf16(float x) {
    uint32_t u;
    std::memcpy(&u, &x, 4);
    if ((u & 0x7f800000u) == 0x7f800000u) return x;
    u = (u + 0x7fffu + ((u >> 16) & 1u)) & 0xffff0000u;
    float r;
    std::memcpy(&r, &u, 4);
    return r;
}

eqs_mlp* mlp_create(int device, hipStream_t stream, const float* params, int bf16, double lr, eqs_ctx* owner) {
    eqs_mlp* n = new eqs_mlp();
    n->device = device;
    n->stream = stream;
    n->owner = owner;
    n->bf16 = bf16 ? 1 : 0;
    const size_t bytes = sizeof(float) * kNParam;
    auto alloc = [&](void** p, size_t nb) {
        if (owner) *p = dev_alloc(owner, nb);
        else EQS_HIP(hipMalloc(p, nb));
    };
    try {
        alloc((void**)&n->master, bytes);
        alloc((void**)&n->wq, bytes);
        alloc((void**)&n->grad, bytes);
        alloc((void**)&n->m1, bytes);
        alloc((void**)&n->m2, bytes);
        alloc((void**)&n->st, sizeof(MlpState));
        std::vector<float> w(params, params + kNParam), wq(kNParam);
        for (int i = 0; i < kNParam; ++i) wq[i] = n->bf16 ? host_bf16(w[i]) : w[i];
        std::vector<float> zero(kNParam, 0.0f);
        EQS_HIP(hipMemcpy(n->master, w.data(), bytes, hipMemcpyHostToDevice));
        EQS_HIP(hipMemcpy(n->wq, wq.data(), bytes, hipMemcpyHostToDevice));
        EQS_HIP(hipMemcpy(n->grad, zero.data(), bytes, hipMemcpyHostToDevice));
        EQS_HIP(hipMemcpy(n->m1, zero.data(), bytes, hipMemcpyHostToDevice));
        EQS_HIP(hipMemcpy(n->m2, zero.data(), bytes, hipMemcpyHostToDevice));
        MlpState s{(float)lr, 0.9f, 0.999f, 1e-8f, 0, 0.0f};
        EQS_HIP(hipMemcpy(n->st, &s, sizeof s, hipMemcpyHostToDevice));
    } catch (...) {
        mlp_destroy(n);
        throw;
    }
    return n;
}

void mlp_destroy(eqs_mlp* n) {
    if (!n) return;
    for (void* p : {(void*)n->master, (void*)n->wq, (void*)n->grad, (void*)n->m1, (void*)n->m2, (void*)n->st}) {
        if (!p) continue;
        if (n->owner) dev_free(n->owner, p);
        else (void)hipFree(p);
    }
    delete n;
}

int64_t mlp_device_bytes() {
    auto r = [](int64_t b) { return (b + 255) / 256 * 256; };
    return 5 * r((int64_t)sizeof(float) * kNParam) + r((int64_t)sizeof(MlpState));
}

void mlp_visit(eqs_mlp* n, const std::function<void(void**)>& f) {
    if (!n) return;
    f((void**)&n->master);
    f((void**)&n->wq);
    f((void**)&n->grad);
    f((void**)&n->m1);
    f((void**)&n->m2);
    f((void**)&n->st);
}

void mlp_forward(eqs_mlp* n, const float* x, float* y, int32_t B) { mlp_launch(n, false, x, nullptr, y, B); }

void mlp_train(eqs_mlp* n, const float* x, const float* t, int32_t B) { mlp_launch(n, true, x, t, nullptr, B); }

void mlp_forward_coeffs(eqs_mlp* n, hipStream_t s, const float* x, const double* P, const double* bias,
                        double* alpha, const double* guard, int32_t* stat) {
    MlpIn in;
    std::memcpy(in.x, x, sizeof in.x);
    std::memcpy(in.P, P, sizeof in.P);
    std::memcpy(in.bias, bias, sizeof in.bias);
    if (n->bf16)
        hipLaunchKernelGGL(k_mlp_alpha<true>, dim3(1), dim3(64), 0, s, in, n->master, n->wq, alpha, guard, stat);
    else
        hipLaunchKernelGGL(k_mlp_alpha<false>, dim3(1), dim3(64), 0, s, in, n->master, n->wq, alpha, guard, stat);
}

void mlp_get(eqs_mlp* n, float* params, float* grad) {
    if (params) EQS_HIP(hipMemcpyAsync(params, n->master, sizeof(float) * kNParam, hipMemcpyDeviceToHost, n->stream));
    if (grad) EQS_HIP(hipMemcpyAsync(grad, n->grad, sizeof(float) * kNParam, hipMemcpyDeviceToHost, n->stream));
    EQS_HIP(hipStreamSynchronize(n->stream));
}

// Checkpoint of the network: master and matmul weights, Adam moments and
// state (the gradient is rewritten by every step). Synchronises its stream.
int64_t mlp_state_bytes() { return (int64_t)(sizeof(float) * 4 * kNParam + sizeof(MlpState)); }
void mlp_save_state(eqs_mlp* n, void* host) {
    char* p = static_cast<char*>(host);
    const size_t b = sizeof(float) * kNParam;
    for (float* src : {n->master, n->wq, n->m1, n->m2}) {
        EQS_HIP(hipMemcpyAsync(p, src, b, hipMemcpyDeviceToHost, n->stream));
        p += b;
    }
    EQS_HIP(hipMemcpyAsync(p, n->st, sizeof(MlpState), hipMemcpyDeviceToHost, n->stream));
    EQS_HIP(hipStreamSynchronize(n->stream));
}
void mlp_load_state(eqs_mlp* n, const void* host) {
    const char* p = static_cast<const char*>(host);
    const size_t b = sizeof(float) * kNParam;
    for (float* dst : {n->master, n->wq, n->m1, n->m2}) {
        EQS_HIP(hipMemcpyAsync(dst, p, b, hipMemcpyHostToDevice, n->stream));
        p += b;
    }
    EQS_HIP(hipMemcpyAsync(n->st, p, sizeof(MlpState), hipMemcpyHostToDevice, n->stream));
    EQS_HIP(hipStreamSynchronize(n->stream));
}

float mlp_last_loss(eqs_mlp* n) {
    MlpState s;
    EQS_HIP(hipMemcpyAsync(&s, n->st, sizeof s, hipMemcpyDeviceToHost, n->stream));
    EQS_HIP(hipStreamSynchronize(n->stream));
    return s.loss;
}

}  // namespace eqs
