// k7: the schedule cost model, a multilayer perceptron in -> 64 -> 64 -> 1
// with ReLU after the two hidden layers, in FP32. It maps features of a
// (circuit, candidate schedule) pair to a predicted log run time; the tuner
// takes the candidate with the smallest prediction. Training minimises the
// mean squared error with Adam (Kingma and Ba, 2015).
//
// Parameters are one flat float array (offsets in mlp_layout):
//   W1[64][in], b1[64], W2[64][64], b2[64], w3[64], b3.
// Inputs are standardised inside the kernels: x' = (x - mean) * inv_std with
// norm = {mean[in], inv_std[in]} (norm may be null: identity).
//
// Samples are counted in int, up to 2^31 - 1 of them: loops go over tiles, and a
// sample's index is formed only where it lies in the batch.
//
// Every reduction runs in a fixed order (matrix products over their inner
// index, per work-group in tile order, across work-groups in group order), so
// results are deterministic for a given batch.
#include <hip/hip_runtime.h>

#include <cmath>
#include <cstdint>

#include "mlp.h"

namespace svk {

namespace {

constexpr int H = kMlpHidden;
constexpr int TILE = 16;        // samples per work-group step: the columns of one matrix instruction
constexpr int THREADS = 256;    // four waves, sixteen hidden units each
constexpr int ROW = TILE + 1;   // LDS row stride [unit][sample]: reads along either index hit 64 different banks
constexpr int MAX_ROWS = 128;   // partial gradients (work-groups of the gradient kernel)

__host__ __device__ constexpr int tiles_of(int batch) { return (batch - 1) / TILE + 1; }

typedef float f4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ float relu(float x) { return x > 0.f ? x : 0.f; }

// 16x16x4 FP32 matrix product: lane 16 q + n gives a = A[n][k_q], b = B[k_q][n]
// and holds D[4 q + r][n] in register r. The order of the k index is free as
// long as both operands use the same: here k = 16 q + s or 4 s + q in step s.
__device__ __forceinline__ f4 mma(float a, float b, f4 c) { return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0); }

// The network on a tile of 16 samples, wave w computing hidden units 16 w ..
// 16 w + 15 of both layers. What a work-group does is a chain of four small
// matrix products with a barrier between them, so it is bound by latency: the
// wave's share of the weights is loaded into registers once per launch (it
// is used for every tile), the activations pass through LDS, and a batch is
// spread over a work-group per 16 samples. One thread per sample, with the
// weights read from LDS for every product, took 259 us for the gradient of
// 128 samples (16 inputs) and 166 us for 4096 predictions.
struct Net {
    MlpLayout L;
    int in, q, n, w;
    float w1[kMlpMaxIn / 4], w2[H / 4];  // A operands: W1[16 w + n][4 s + q], W2[16 w + n][16 q + s]
    float b1[4], b2[4], w3[4], b3;       // of units 16 w + 4 q + r

    __device__ __forceinline__ void load(const float *P, int in_)
    {
        in = in_;
        L = mlp_layout(in);
        const int lane = threadIdx.x & 63;
        q = lane >> 4;
        n = lane & 15;
        w = threadIdx.x >> 6;
        const int row = 16 * w + n;
#pragma unroll
        for (int s = 0; s < kMlpMaxIn / 4; ++s) w1[s] = 4 * s + q < in ? P[L.w1 + row * in + 4 * s + q] : 0.f;
#pragma unroll
        for (int s = 0; s < H / 4; ++s) w2[s] = P[L.w2 + row * H + 16 * q + s];
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            b1[r] = P[L.b1 + unit(r)];
            b2[r] = P[L.b2 + unit(r)];
            w3[r] = P[L.w3 + unit(r)];
        }
        b3 = P[L.b3];
    }
    __device__ __forceinline__ int unit(int r) const { return 16 * w + 4 * q + r; }

    // Standardised inputs of samples s0 .. s0 + 15 as xs[input][sample], zeros beyond the `left` samples from s0 on
    // and the inputs.
    __device__ __forceinline__ void stage(float (*xs)[ROW], const float *X, const float *norm, int s0, int left) const
    {
        for (int e = threadIdx.x; e < TILE * kMlpMaxIn; e += THREADS) {
            const int i = e % kMlpMaxIn, s = e / kMlpMaxIn;
            float x = 0.f;
            if (i < in && s < left) {
                x = X[(size_t)(s0 + s) * in + i];
                if (norm) x = (x - norm[i]) * norm[in + i];
            }
            xs[i][s] = x;
        }
    }
    // Forward pass of the staged tile: this wave's units of h1 and h2 (zero where sample n is not valid), all of
    // h1 in h1s; returns y of sample n.
    __device__ __forceinline__ float forward(const float (*xs)[ROW], float (*h1s)[ROW], float (*ys)[TILE], bool valid,
                                             f4 &h1, f4 &h2) const
    {
        f4 a = {b1[0], b1[1], b1[2], b1[3]};
#pragma unroll
        for (int s = 0; s < kMlpMaxIn / 4; ++s)
            if (4 * s < in) a = mma(w1[s], xs[4 * s + q][n], a);
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            h1[r] = valid ? relu(a[r]) : 0.f;
            h1s[unit(r)][n] = h1[r];
        }
        __syncthreads();
        f4 c = {b2[0], b2[1], b2[2], b2[3]};
#pragma unroll
        for (int s = 0; s < H / 4; ++s) c = mma(w2[s], h1s[16 * q + s][n], c);
        float y = 0.f;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            h2[r] = valid ? relu(c[r]) : 0.f;
            y = fmaf(w3[r], h2[r], y);
        }
        y += __shfl_xor(y, 16, 64);
        y += __shfl_xor(y, 32, 64);
        if (q == 0) ys[w][n] = y;
        __syncthreads();
        return b3 + ((ys[0][n] + ys[1][n]) + (ys[2][n] + ys[3][n]));
    }
};

// Predictions, tiles of 16 samples grid-stride. With argmin (one work-group)
// also the index of the smallest.
__global__ void __launch_bounds__(THREADS) k7_forward_kernel(const float *P, int in, const float *norm,
                                                             const float *X, int batch, float *y, int *argmin)
{
    __shared__ float xs[kMlpMaxIn][ROW], h1s[H][ROW], ys[4][TILE], all[kMlpArgminMax];
    Net net;
    net.load(P, in);
    for (int t = blockIdx.x; t < tiles_of(batch); t += gridDim.x) {
        const int s0 = t * TILE, left = batch - s0;
        net.stage(xs, X, norm, s0, left);
        __syncthreads();
        f4 h1, h2;
        const bool valid = net.n < left;
        const float out = net.forward(xs, h1s, ys, valid, h1, h2);
        if (threadIdx.x < TILE && valid) {
            y[s0 + net.n] = out;
            if (argmin) all[s0 + net.n] = out;
        }
        __syncthreads();
    }
    if (argmin && threadIdx.x == 0) {
        int best = 0;
        for (int k = 1; k < batch; ++k)
            if (all[k] < all[best]) best = k;
        *argmin = best;
    }
}

// Gradient of the mean squared error over the batch. A work-group takes
// tiles of 16 samples (grid-stride), keeps its share of the gradient in
// registers (as matrix accumulators for W1 and W2) and writes one partial row
// of count + 1 floats (last: loss).
__global__ void __launch_bounds__(THREADS) k7_grad_kernel(const float *P, int in, const float *norm,
                                                          const float *X, const float *T, int batch, float *partial)
{
    __shared__ float xs[kMlpMaxIn][ROW], h1s[H][ROW], d1s[H][ROW], d2s[H][ROW], ys[4][TILE];
    Net net;
    net.load(P, in);
    const int q = net.q, n = net.n, w = net.w;
    float w2t[H / 4];  // A operand of W2^T: W2[16 q + s][16 w + n]
#pragma unroll
    for (int s = 0; s < H / 4; ++s) w2t[s] = P[net.L.w2 + (16 * q + s) * H + 16 * w + n];
    const float inv_b = 1.f / (float)batch;
    const f4 zero = {0.f, 0.f, 0.f, 0.f};
    f4 g1[kMlpMaxIn / 16] = {zero, zero}, g2[4] = {zero, zero, zero, zero};
    f4 gb1 = zero, gb2 = zero, gw3 = zero;
    float gb3 = 0.f, loss = 0.f;
    for (int t = blockIdx.x; t < tiles_of(batch); t += gridDim.x) {
        const int s0 = t * TILE, left = batch - s0;
        net.stage(xs, X, norm, s0, left);
        const bool valid = n < left;
        const float target = valid ? T[s0 + n] : 0.f;
        __syncthreads();
        f4 h1, h2, d2;
        const float yv = net.forward(xs, h1s, ys, valid, h1, h2);
        const float r = valid ? yv - target : 0.f;
        const float dy = 2.f * r * inv_b;
        loss += r * r;
        gb3 += dy;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            d2[j] = h2[j] > 0.f ? dy * net.w3[j] : 0.f;
            d2s[net.unit(j)][n] = d2[j];
            gb2[j] += d2[j];
            gw3[j] = fmaf(dy, h2[j], gw3[j]);
        }
        __syncthreads();
        f4 d1 = zero;
#pragma unroll
        for (int s = 0; s < H / 4; ++s) d1 = mma(w2t[s], d2s[16 * q + s][n], d1);
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            if (!(h1[j] > 0.f)) d1[j] = 0.f;
            d1s[net.unit(j)][n] = d1[j];
            gb1[j] += d1[j];
        }
        // W2[16 w ..][16 c ..] += d2 h1^T, W1 += d1 x^T over the tile's samples (k = 4 s + q)
#pragma unroll
        for (int s = 0; s < TILE / 4; ++s) {
            const float a = d2s[16 * w + n][4 * s + q];
#pragma unroll
            for (int c = 0; c < 4; ++c) g2[c] = mma(a, h1s[16 * c + n][4 * s + q], g2[c]);
        }
        __syncthreads();
#pragma unroll
        for (int s = 0; s < TILE / 4; ++s) {
            const float a = d1s[16 * w + n][4 * s + q];
#pragma unroll
            for (int c = 0; c < kMlpMaxIn / 16; ++c)
                if (16 * c < in) g1[c] = mma(a, xs[16 * c + n][4 * s + q], g1[c]);
        }
        __syncthreads();
    }
    // sums over the samples a wave's 16 columns hold
    auto cols = [](float v) {
#pragma unroll
        for (int b = 1; b < 16; b <<= 1) v += __shfl_xor(v, b, 64);
        return v;
    };
    const MlpLayout &L = net.L;
    float *row = partial + (size_t)blockIdx.x * (L.count + 1);
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const int u = net.unit(j);
#pragma unroll
        for (int c = 0; c < kMlpMaxIn / 16; ++c)
            if (16 * c + n < in) row[L.w1 + u * in + 16 * c + n] = g1[c][j];
#pragma unroll
        for (int c = 0; c < 4; ++c) row[L.w2 + u * H + 16 * c + n] = g2[c][j];
        const float vb1 = cols(gb1[j]), vb2 = cols(gb2[j]), vw3 = cols(gw3[j]);
        if (n == 0) {
            row[L.b1 + u] = vb1;
            row[L.b2 + u] = vb2;
            row[L.w3 + u] = vw3;
        }
    }
    const float vb3 = cols(gb3), vl = cols(loss);
    if (threadIdx.x == 0) {
        row[L.b3] = vb3;
        row[L.count] = vl * inv_b;
    }
}

// Sum of the partial rows in group order: grad[e] and, at e == count, loss.
__global__ void __launch_bounds__(256) k7_reduce_kernel(const float *partial, int groups, int count, float *grad,
                                                        float *loss)
{
    const int e = blockIdx.x * blockDim.x + threadIdx.x;
    if (e > count) return;
    float t = 0.f;
#pragma unroll 8
    for (int g = 0; g < groups; ++g) t += partial[(size_t)g * (count + 1) + e];
    if (e < count) grad[e] = t;
    else if (loss) *loss = t;
}

// Adam with bias correction: c1 = 1 - beta1^step, c2 = 1 - beta2^step, formed
// on the host (two FP64 powers per thread took most of this kernel's time).
__global__ void __launch_bounds__(256) k7_adam_kernel(float *P, float *m, float *v, const float *g, int count,
                                                      float lr, float beta1, float beta2, float eps, double c1, double c2)
{
    const int e = blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= count) return;
    const float ge = g[e];
    const float me = beta1 * m[e] + (1.f - beta1) * ge;
    const float ve = beta2 * v[e] + (1.f - beta2) * ge * ge;
    m[e] = me;
    v[e] = ve;
    const float mh = (float)(me / c1);
    const float vh = (float)(ve / c2);
    P[e] -= lr * mh / (sqrtf(vh) + eps);
}

bool in_ok(int in) { return in >= 1 && in <= kMlpMaxIn; }

}  // namespace

int mlp_grad_groups(int batch)
{
    const int tiles = tiles_of(batch);
    return tiles < MAX_ROWS ? tiles : MAX_ROWS;
}

hipError_t mlp_forward(const float *P, int in, const float *norm, const float *X, int batch, float *y,
                       int *argmin, hipStream_t st)
{
    if (!in_ok(in) || batch < 1) return hipErrorInvalidValue;
    if (argmin && batch > kMlpArgminMax) return hipErrorInvalidValue;
    // a work-group per tile up to four per CU, which then take several tiles each
    const int tiles = tiles_of(batch);
    const unsigned grid = argmin ? 1u : (unsigned)(tiles < 1024 ? tiles : 1024);
    k7_forward_kernel<<<grid, THREADS, 0, st>>>(P, in, norm, X, batch, y, argmin);
    return hipGetLastError();
}

hipError_t mlp_grad(const float *P, int in, const float *norm, const float *X, const float *T, int batch,
                    float *grad, float *loss, float *workspace, hipStream_t st)
{
    if (!in_ok(in) || batch < 1) return hipErrorInvalidValue;
    const MlpLayout L = mlp_layout(in);
    const int groups = mlp_grad_groups(batch);
    k7_grad_kernel<<<groups, THREADS, 0, st>>>(P, in, norm, X, T, batch, workspace);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    k7_reduce_kernel<<<(L.count + 1 + 255) / 256, 256, 0, st>>>(workspace, groups, L.count, grad, loss);
    return hipGetLastError();
}

hipError_t mlp_adam(float *P, float *m, float *v, const float *g, int count, float lr, float beta1, float beta2,
                    float eps, int step, hipStream_t st)
{
    if (count < 1 || step < 1) return hipErrorInvalidValue;
    const double c1 = 1.0 - std::pow((double)beta1, (double)step), c2 = 1.0 - std::pow((double)beta2, (double)step);
    k7_adam_kernel<<<(count + 255) / 256, 256, 0, st>>>(P, m, v, g, count, lr, beta1, beta2, eps, c1, c2);
    return hipGetLastError();
}

}  // namespace svk
