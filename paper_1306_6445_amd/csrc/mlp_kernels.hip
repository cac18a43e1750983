// Training and inference kernels of the 3-64-64-3 tanh surrogate network
// (declared in include/lbm_mlp.h).
//
// A workgroup of 512 threads (eight wave64s) takes chunks of 16 samples: the
// parameters, the chunk's inputs and both hidden layers sit in LDS, so one
// launch runs the whole forward pass and backpropagation, and each workgroup
// writes the gradient of its chunks (plus its share of the loss) to its slot.  A
// second kernel sums the slots in a fixed order and applies the Adam update, so
// results do not depend on scheduling.
//
// A training step is bound by latency, not by its 37 MFLOP: the chunk decides
// how many CUs share the batch and how long each one's chain is.  At 1,392 rows
// 87 workgroups of 16 samples take 9 us where 44 of 32 samples (256 threads)
// took 26, and the Adam kernel, whose threads summed 44 slots one after the
// other, takes 4 us with 16 threads to a parameter instead of 12.
//
// Thread mapping: for [sample][unit] arrays the 64 lanes of a wave take the 64
// units and the wave takes two samples at a time, so each weight read from LDS
// serves both and the samples' activations are broadcast, four to a read.  W2
// has a row stride of 65 floats (lanes that walk a column hit 64 different
// banks), the activations one of 68 (16-byte rows; the 16 lanes that walk a
// column hit 16 banks).  The working set is about 37 KB.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "mlp_kernels.hpp"

namespace lbm {
namespace mlp {

constexpr int CH = 16;         // samples of a chunk
constexpr int NT = 512;        // threads per workgroup
constexpr int NW = NT / H;     // waves
constexpr int LDW = H + 1;     // row stride of W2
constexpr int LDA = H + 4;     // row stride of the activation arrays
constexpr int MAX_SLOTS = 512; // gradient slots: two workgroups a CU
static_assert(CH == 2 * NW, "each wave takes two samples of a chunk");

struct Smem {
    float h1[CH * LDA], h2[CH * LDA], dz2[CH * LDA], dz1[CH * LDA];
    float W1[H * IN], b1[H], W2[H * LDW], b2[H], W3[OUT * H], b3[4];
    float x[CH * IN];
    float dy[OUT * CH];  // [k][s]
    double red[H];
};

__device__ __forceinline__ void load_params(Smem &S, const float *__restrict__ th)
{
    const int t = threadIdx.x;
    for (int i = t; i < H * IN; i += NT) S.W1[i] = th[OFF_W1 + i];
    for (int i = t; i < H; i += NT) {
        S.b1[i] = th[OFF_B1 + i];
        S.b2[i] = th[OFF_B2 + i];
    }
#pragma unroll
    for (int i = 0; i < H * H / NT; ++i) S.W2[((t + i * NT) / H) * LDW + t % H] = th[OFF_W2 + t + i * NT];
    for (int i = t; i < OUT * H; i += NT) S.W3[i] = th[OFF_W3 + i];
    if (t < OUT) S.b3[t] = th[OFF_B3 + t];
}

// Inputs of the chunk starting at sample s0 (rows past n are zero).
__device__ __forceinline__ void load_inputs(Smem &S, const float *__restrict__ x, int64_t s0, int n)
{
    const int i = threadIdx.x;
    if (i < CH * IN) S.x[i] = s0 + i / IN < n ? x[s0 * IN + i] : 0.0f;
}

// z = b2[j] + sum_k W2[j][k] in[k] for the wave's two samples (before the tanh).
__device__ __forceinline__ void hidden2(const Smem &S, const float *in0, const float *in1, int j, float &z0, float &z1)
{
    z0 = z1 = S.b2[j];
#pragma unroll 4
    for (int k = 0; k < H; k += 4) {
        const float4 a = *reinterpret_cast<const float4 *>(in0 + k), b = *reinterpret_cast<const float4 *>(in1 + k);
        const float *w = S.W2 + j * LDW + k;
        z0 += w[0] * a.x;
        z1 += w[0] * b.x;
        z0 += w[1] * a.y;
        z1 += w[1] * b.y;
        z0 += w[2] * a.z;
        z1 += w[2] * b.z;
        z0 += w[3] * a.w;
        z1 += w[3] * b.w;
    }
}

// Both hidden layers of the chunk into S.h1 and S.h2.  A wave reads back only
// the rows that it wrote.
__device__ __forceinline__ void hidden_layers(Smem &S)
{
    const int j = threadIdx.x & (H - 1), s = 2 * (threadIdx.x >> 6);
    float z0 = S.b1[j], z1 = z0;
#pragma unroll
    for (int i = 0; i < IN; ++i) {
        const float w = S.W1[j * IN + i];
        z0 += w * S.x[s * IN + i];
        z1 += w * S.x[(s + 1) * IN + i];
    }
    float *r0 = S.h1 + s * LDA, *r1 = r0 + LDA;
    r0[j] = tanhf(z0);
    r1[j] = tanhf(z1);
    __syncthreads();
    hidden2(S, r0, r1, j, z0, z1);
    S.h2[s * LDA + j] = tanhf(z0);
    S.h2[(s + 1) * LDA + j] = tanhf(z1);
    __syncthreads();
}

// Output k of sample s (threads 0..47: k = t / 16, s = t % 16).
__device__ __forceinline__ float output_unit(const Smem &S, int k, int s)
{
    float y = S.b3[k];
#pragma unroll 16
    for (int j = 0; j < H; ++j) y += S.W3[k * H + j] * S.h2[s * LDA + j];
    return y;
}

__global__ void __launch_bounds__(NT) forward_kernel(const float *__restrict__ th, const float *__restrict__ x, int n,
                                                     float *__restrict__ y)
{
    __shared__ __align__(16) Smem S;
    load_params(S, th);
    for (int64_t s0 = (int64_t)blockIdx.x * CH; s0 < n; s0 += (int64_t)gridDim.x * CH) {
        load_inputs(S, x, s0, n);
        __syncthreads();
        hidden_layers(S);
        const int t = threadIdx.x;
        if (t < OUT * CH) {
            const int k = t / CH, s = t % CH;
            if (s0 + s < n) y[(s0 + s) * OUT + k] = output_unit(S, k, s);
        }
        __syncthreads();
    }
}

// Sum of the weights m over all entries -> inv[0] = 1 / sum (0 when the sum is 0).
constexpr int WS = 256;
__global__ void __launch_bounds__(WS) weight_sum_kernel(const float *__restrict__ m, int n, float *__restrict__ inv)
{
    __shared__ double red[WS];
    double acc = 0.0;
    for (int64_t i = threadIdx.x; i < (int64_t)n * OUT; i += WS) acc += (double)m[i];
    red[threadIdx.x] = acc;
    __syncthreads();
    for (unsigned o = WS / 2; o > 0; o >>= 1) {
        if (threadIdx.x < o) red[threadIdx.x] += red[threadIdx.x + o];
        __syncthreads();
    }
    if (threadIdx.x == 0) inv[0] = red[0] > 0.0 ? (float)(1.0 / red[0]) : 0.0f;
}

// Loss share and gradient of the workgroup's chunks: partial[blockIdx.x][P], ploss[blockIdx.x].
__global__ void __launch_bounds__(NT) grad_kernel(const float *__restrict__ th, const float *__restrict__ x,
                                                  const float *__restrict__ tg, const float *__restrict__ mw, int n,
                                                  const float *__restrict__ inv_wsum, float *__restrict__ partial,
                                                  double *__restrict__ ploss)
{
    __shared__ __align__(16) Smem S;
    const int t = threadIdx.x, lane = t & (H - 1), w = t >> 6, s = 2 * w;
    const float iw = inv_wsum[0];
    load_params(S, th);
    // the workgroup's sums: dW2[NW w + i][lane], one entry of dW3 and b3, of dW1 and b1, of b2, the loss (in FP64:
    // past MAX_SLOTS chunks a thread adds one term of each of its chunks)
    float g2[H / NW] = {}, g3 = 0.0f, g1 = 0.0f, gb2 = 0.0f;
    double lsum = 0.0;
    for (int64_t s0 = (int64_t)blockIdx.x * CH; s0 < n; s0 += (int64_t)gridDim.x * CH) {
        load_inputs(S, x, s0, n);
        __syncthreads();
        hidden_layers(S);

        // dL/dy = m (y - t) / sum(m); loss share m (y - t)^2 / (2 sum(m))
        if (t < OUT * CH) {
            const int k = t / CH, q = t % CH;
            float d = 0.0f;
            if (s0 + q < n) {
                const int64_t e = (s0 + q) * OUT + k;
                const float r = output_unit(S, k, q) - tg[e];
                const float mr = mw[e] * r;
                d = mr * iw;
                const float share = 0.5f * iw * (mr * r);
                lsum += (double)share;
            }
            S.dy[k * CH + q] = d;
        }
        __syncthreads();

        // output layer: dW3[k][j] = sum_s dy[k][s] h2[s][j], db3[k] = sum_s dy[k][s]
        if (t < OUT * H) {
#pragma unroll
            for (int q = 0; q < CH; ++q) g3 += S.dy[w * CH + q] * S.h2[q * LDA + lane];
        } else if (t < OUT * H + OUT) {
            for (int q = 0; q < CH; ++q) g3 += S.dy[(t - OUT * H) * CH + q];
        }
        // through tanh: dz2[s][j] = (sum_k W3[k][j] dy[k][s]) (1 - h2[s][j]^2)
#pragma unroll
        for (int q = s; q < s + 2; ++q) {
            float a = 0.0f;
#pragma unroll
            for (int k = 0; k < OUT; ++k) a += S.W3[k * H + lane] * S.dy[k * CH + q];
            const float h = S.h2[q * LDA + lane];
            S.dz2[q * LDA + lane] = a * (1.0f - h * h);
        }
        __syncthreads();

        // hidden layer 2: dW2[j][k] = sum_s dz2[s][j] h1[s][k], db2[j] = sum_s dz2[s][j]
#pragma unroll 4
        for (int q = 0; q < CH; ++q) {
            const float h = S.h1[q * LDA + lane];
            const float4 a = *reinterpret_cast<const float4 *>(&S.dz2[q * LDA + w * (H / NW)]),
                         b = *reinterpret_cast<const float4 *>(&S.dz2[q * LDA + w * (H / NW) + 4]);
            g2[0] += a.x * h;
            g2[1] += a.y * h;
            g2[2] += a.z * h;
            g2[3] += a.w * h;
            g2[4] += b.x * h;
            g2[5] += b.y * h;
            g2[6] += b.z * h;
            g2[7] += b.w * h;
        }
        if (t < H)
            for (int q = 0; q < CH; ++q) gb2 += S.dz2[q * LDA + t];
        // dz1[s][k] = (sum_j W2[j][k] dz2[s][j]) (1 - h1[s][k]^2)
        {
            const float *d0 = S.dz2 + s * LDA, *d1 = d0 + LDA;
            float a0 = 0.0f, a1 = 0.0f;
#pragma unroll 4
            for (int j = 0; j < H; j += 4) {
                const float4 p = *reinterpret_cast<const float4 *>(d0 + j), q = *reinterpret_cast<const float4 *>(d1 + j);
                const float w0 = S.W2[j * LDW + lane], w1 = S.W2[(j + 1) * LDW + lane], w2 = S.W2[(j + 2) * LDW + lane],
                            w3 = S.W2[(j + 3) * LDW + lane];
                a0 += w0 * p.x;
                a1 += w0 * q.x;
                a0 += w1 * p.y;
                a1 += w1 * q.y;
                a0 += w2 * p.z;
                a1 += w2 * q.z;
                a0 += w3 * p.w;
                a1 += w3 * q.w;
            }
            const float h0 = S.h1[s * LDA + lane], h1 = S.h1[(s + 1) * LDA + lane];
            S.dz1[s * LDA + lane] = a0 * (1.0f - h0 * h0);
            S.dz1[(s + 1) * LDA + lane] = a1 * (1.0f - h1 * h1);
        }
        __syncthreads();

        // hidden layer 1: dW1[j][i] = sum_s dz1[s][j] x[s][i], db1[j] = sum_s dz1[s][j]
        if (t < IN * H) {
#pragma unroll
            for (int q = 0; q < CH; ++q) g1 += S.dz1[q * LDA + lane] * S.x[q * IN + w];
        } else if (t < IN * H + H) {
            for (int q = 0; q < CH; ++q) g1 += S.dz1[q * LDA + lane];
        }
        __syncthreads();
    }

    float *g = partial + (int64_t)blockIdx.x * P;
#pragma unroll
    for (int i = 0; i < H / NW; ++i) g[OFF_W2 + (w * (H / NW) + i) * H + lane] = g2[i];
    if (t < OUT * H)
        g[OFF_W3 + t] = g3;
    else if (t < OUT * H + OUT)
        g[OFF_B3 + t - OUT * H] = g3;
    if (t < H) g[OFF_B2 + t] = gb2;
    if (t < IN * H)
        g[OFF_W1 + lane * IN + w] = g1;
    else if (t < IN * H + H)
        g[OFF_B1 + lane] = g1;
    // the loss share (only the first OUT * CH threads hold one)
    if (t < H) S.red[t] = lsum;
    __syncthreads();
    for (int o = H / 2; o > 0; o >>= 1) {
        if (t < o) S.red[t] += S.red[t + o];
        __syncthreads();
    }
    if (t == 0) ploss[blockIdx.x] = S.red[0];
}
static_assert(OUT * CH <= H, "the loss reduction spans one wave's threads");

// Sum of the gradient slots (fixed order: AG threads a parameter take every
// AG-th slot, then their sums in order); optionally the Adam update
//   m <- b1 m + (1 - b1) g, v <- b2 v + (1 - b2) g^2,
//   theta <- theta - lr (c1 m) / (sqrt(c2 v) + eps),  c1 = 1/(1-b1^t), c2 = 1/(1-b2^t).
constexpr int AG = 16, AP = 32; // threads a parameter, parameters a workgroup
__global__ void __launch_bounds__(AG *AP) adam_kernel(float *__restrict__ th, float *__restrict__ m1,
                                                      float *__restrict__ m2, const float *__restrict__ partial,
                                                      int nch, float *__restrict__ grad, AdamArgs a)
{
    __shared__ float red[AG][AP];
    const int i = threadIdx.x % AP, q = threadIdx.x / AP, p = blockIdx.x * AP + i;
    float g = 0.0f;
    if (p < P) {
#pragma unroll 8
        for (int c = q; c < nch; c += AG) g += partial[(int64_t)c * P + p];
    }
    red[q][i] = g;
    __syncthreads();
    if (q > 0 || p >= P) return;
    g = 0.0f;
#pragma unroll
    for (int c = 0; c < AG; ++c) g += red[c][i];
    if (grad) grad[p] = g;
    if (!a.update) return;
    const float m = a.beta1 * m1[p] + (1.0f - a.beta1) * g;
    const float v = a.beta2 * m2[p] + (1.0f - a.beta2) * (g * g);
    m1[p] = m;
    m2[p] = v;
    th[p] -= a.lr * (a.c1 * m) / (sqrtf(a.c2 * v) + a.eps);
}

int chunks(int n) { return n > CH * MAX_SLOTS ? MAX_SLOTS : (n + CH - 1) / CH; }

hipError_t launch_forward(const float *th, const float *x, int n, float *y, hipStream_t st)
{
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(forward_kernel, dim3(chunks(n)), dim3(NT), 0, st, th, x, n, y);
    return hipGetLastError();
}

hipError_t launch_weight_sum(const float *m, int n, float *inv, hipStream_t st)
{
    hipLaunchKernelGGL(weight_sum_kernel, dim3(1), dim3(WS), 0, st, m, n, inv);
    return hipGetLastError();
}

hipError_t launch_grad(const float *th, const float *x, const float *tg, const float *mw, int n, const float *inv,
                       float *partial, double *ploss, hipStream_t st)
{
    hipLaunchKernelGGL(grad_kernel, dim3(chunks(n)), dim3(NT), 0, st, th, x, tg, mw, n, inv, partial,
                       ploss);
    return hipGetLastError();
}

hipError_t launch_adam(float *th, float *m1, float *m2, const float *partial, int nch, float *grad, const AdamArgs &a,
                       hipStream_t st)
{
    hipLaunchKernelGGL(adam_kernel, dim3((P + AP - 1) / AP), dim3(AG * AP), 0, st, th, m1, m2, partial, nch, grad, a);
    return hipGetLastError();
}

} // namespace mlp
} // namespace lbm
