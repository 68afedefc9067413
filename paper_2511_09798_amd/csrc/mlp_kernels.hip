// mlp_kernels.hip -- the learned predictor's network on gfx950, FP32: a
// 24-128-128-128-2 multilayer perceptron with tanh hidden layers, its
// back-propagation, the weighted mean squared error and Adam.  Parameters are
// flat, layer by layer: W_l (out x in, row-major) then b_l.  Batches are
// row-major (sample-major).  All reductions run in a fixed order, so
// training is deterministic.
#include <math.h>

#include "kernels.hpp"

namespace mqh {

static_assert(kMlpLayers == 4 && kMlpWidth == 128 && kMlpOut == 2 && kMlpIn <= 32, "layout of the fused kernels");

// Offset of layer l's weights in the parameters (its biases follow the weights).
__host__ __device__ constexpr int64_t mlp_off(int l) {
    int64_t off = 0;
    for (int q = 0; q < l; ++q) {
        const int in = q == 0 ? kMlpIn : kMlpWidth, out = q == kMlpLayers - 1 ? kMlpOut : kMlpWidth;
        off += (int64_t)out * in + out;
    }
    return off;
}

// ---------------------------------------------------------------------------
// The network is 73 KFLOP a sample: a batch's step is bound by launches and
// memory latencies, so each direction is one or two launches.  All
// contractions run on the FP32 matrix cores (v_mfma_f32_16x16x4_f32: lane l
// supplies A[l%16][l/16] and B[l/16][l%16] and receives D[4(l/16) + r][l%16]).
// As one 64 x 64-tile GEMM per layer and direction and serial column sums (17
// launches of 4 .. 50 us on 2 .. 8 workgroups) a training step took 532 us on
// 256 samples and 3.18 ms on 2 048; in these 5 launches 29 and 79 us.
// ---------------------------------------------------------------------------

typedef float v4f __attribute__((ext_vector_type(4)));
constexpr int kMlpRows = 16;             // samples per workgroup of the fused kernels
constexpr int kMlpLd = kMlpWidth + 4;    // padded LDS row

// Four consecutive parameters (VEC: 16-byte aligned).
template <bool VEC>
__device__ __forceinline__ v4f load4(const float* __restrict__ p) {
    if (VEC) return *reinterpret_cast<const v4f*>(p);
    v4f v;
    v[0] = p[0];
    v[1] = p[1];
    v[2] = p[2];
    v[3] = p[3];
    return v;
}

// y and the tanh outputs of 16 samples through all four layers.  Wave w of eight
// forms columns 16 w .. + 15 of a hidden layer; contraction step s takes k =
// 16 s + 4 (l/16) + j in its j-th product, so a lane reads four consecutive
// weights of an output row.  Every weight a lane needs is loaded before the
// first layer starts (18 float4), which leaves one memory latency instead of
// four.
constexpr int kMlpThreads = 512;
static_assert(kMlpThreads / kWave * 16 == kMlpWidth, "one 16-column tile per wave");

template <int STEPS>
__device__ __forceinline__ void mlp_layer(const float (*in)[kMlpLd], float (*out)[kMlpLd], const v4f (&wt)[STEPS],
                                          float bias, int B, int64_t b0, float* __restrict__ hid) {
    const int lane = threadIdx.x & (kWave - 1), li = lane & 15, lk = lane >> 4;
    const int n = 16 * (threadIdx.x / kWave) + li;
    v4f acc = v4f{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int s = 0; s < STEPS; ++s) {
        const v4f h = *reinterpret_cast<const v4f*>(&in[li][16 * s + 4 * lk]);
#pragma unroll
        for (int j = 0; j < 4; ++j) acc = __builtin_amdgcn_mfma_f32_16x16x4f32(h[j], wt[s][j], acc, 0, 0, 0);
    }
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const int row = 4 * lk + r;
        const float v = tanhf(acc[r] + bias);
        out[row][n] = v;
        if (b0 + row < B) hid[(b0 + row) * kMlpWidth + n] = v;
    }
    __syncthreads();
}

template <bool VEC>
__global__ __launch_bounds__(kMlpThreads) void k_mlp_forward(const float* __restrict__ params,
                                                             const float* __restrict__ x, int B,
                                                             float* __restrict__ y, float* __restrict__ hidden) {
    __shared__ float H[2][kMlpRows][kMlpLd];
    const int tid = threadIdx.x, lane = tid & (kWave - 1);
    const int li = lane & 15, lk = lane >> 4;
    const int n = 16 * (tid / kWave) + li;
    const int64_t b0 = (int64_t)blockIdx.x * kMlpRows;
    const int64_t hs = (int64_t)B * kMlpWidth;  // a layer's block of activations
    v4f w0[2], w1[8], w2[8];
#pragma unroll
    for (int s = 0; s < 2; ++s) {
        const int k = 16 * s + 4 * lk;
        w0[s] = k < kMlpIn ? load4<VEC>(params + (int64_t)n * kMlpIn + k) : v4f{0.f, 0.f, 0.f, 0.f};
    }
#pragma unroll
    for (int s = 0; s < 8; ++s) {
        w1[s] = load4<VEC>(params + mlp_off(1) + (int64_t)n * kMlpWidth + 16 * s + 4 * lk);
        w2[s] = load4<VEC>(params + mlp_off(2) + (int64_t)n * kMlpWidth + 16 * s + 4 * lk);
    }
    const float c0 = params[mlp_off(0) + kMlpWidth * kMlpIn + n];
    const float c1 = params[mlp_off(1) + kMlpWidth * kMlpWidth + n];
    const float c2 = params[mlp_off(2) + kMlpWidth * kMlpWidth + n];
    if (tid < kMlpRows * 32) {
        const int r = tid / 32, k = tid % 32;
        H[0][r][k] = k < kMlpIn && b0 + r < B ? x[(b0 + r) * kMlpIn + k] : 0.f;
    }
    __syncthreads();
    mlp_layer<2>(H[0], H[1], w0, c0, B, b0, hidden);
    mlp_layer<8>(H[1], H[0], w1, c1, B, b0, hidden + hs);
    mlp_layer<8>(H[0], H[1], w2, c2, B, b0, hidden + 2 * hs);
    // 32 outputs, sixteen lanes each
    const int o = tid >> 4, q = tid & 15, row = o >> 1, k = o & 1;
    const float* w3 = params + mlp_off(3) + k * kMlpWidth + 8 * q;
    float v = 0.f;
#pragma unroll
    for (int e = 0; e < 8; ++e) v = fmaf(H[1][row][8 * q + e], w3[e], v);
    v += __shfl_xor(v, 1, kWave);
    v += __shfl_xor(v, 2, kWave);
    v += __shfl_xor(v, 4, kWave);
    v += __shfl_xor(v, 8, kWave);
    if (q == 0 && b0 + row < B) y[(b0 + row) * kMlpOut + k] = v + params[mlp_off(3) + kMlpOut * kMlpWidth + k];
}

// dL/dz of layer 2 for one sample and column (rank two in dy): (dy W_3) (1 - h^2).
__device__ __forceinline__ float dz_out(float d0, float d1, float wa, float wb, float h) {
    return fmaf(d0, wa, d1 * wb) * (1.f - h * h);
}

// dL/dz of layers 1 and 0 for 16 samples (dz1, dz0: batch x 128 each); layer
// 2's follows from dy and is not stored.  Lanes and columns as in the forward
// kernel; the weights are read transposed (B[k][n] = W[k][n]), both layers'
// before the first product.
__global__ __launch_bounds__(kMlpThreads) void k_mlp_data_grad(const float* __restrict__ params,
                                                               const float* __restrict__ hidden,
                                                               const float* __restrict__ dy, int B,
                                                               float* __restrict__ dz1, float* __restrict__ dz0) {
    __shared__ float D[2][kMlpRows][kMlpLd];
    const int tid = threadIdx.x, lane = tid & (kWave - 1);
    const int li = lane & 15, lk = lane >> 4;
    const int n = 16 * (tid / kWave) + li;
    const int64_t b0 = (int64_t)blockIdx.x * kMlpRows;
    const int64_t hs = (int64_t)B * kMlpWidth;
    float wt[2][kMlpWidth / 4];
#pragma unroll
    for (int l = 1; l >= 0; --l) {
        const float* W = params + mlp_off(l + 1) + n;
#pragma unroll
        for (int e = 0; e < kMlpWidth / 4; ++e) wt[l][e] = W[(16 * (e / 4) + 4 * lk + e % 4) * kMlpWidth];
    }
    const float* w3 = params + mlp_off(3);
#pragma unroll
    for (int e = tid; e < kMlpRows * kMlpWidth; e += kMlpThreads) {
        const int r = e / kMlpWidth, i = e % kMlpWidth;
        const int64_t b = b0 + r < B ? b0 + r : B - 1;
        const float v = dz_out(dy[b * kMlpOut], dy[b * kMlpOut + 1], w3[i], w3[kMlpWidth + i],
                               hidden[2 * hs + b * kMlpWidth + i]);
        D[0][r][i] = b0 + r < B ? v : 0.f;
    }
    __syncthreads();
#pragma unroll
    for (int l = 1; l >= 0; --l) {  // dz of layer l from that of layer l + 1
        const float(*in)[kMlpLd] = D[1 - l];
        float* dz = l == 1 ? dz1 : dz0;
        v4f acc = v4f{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int s = 0; s < kMlpWidth / 16; ++s) {
            const v4f d = *reinterpret_cast<const v4f*>(&in[li][16 * s + 4 * lk]);
#pragma unroll
            for (int j = 0; j < 4; ++j) acc = __builtin_amdgcn_mfma_f32_16x16x4f32(d[j], wt[l][4 * s + j], acc, 0, 0, 0);
        }
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int row = 4 * lk + r;
            const int64_t b = b0 + row;
            float v = 0.f;
            if (b < B) {
                const float h = hidden[l * hs + b * kMlpWidth + n];
                v = acc[r] * (1.f - h * h);
                dz[b * kMlpWidth + n] = v;
            }
            if (l == 1) D[1][row][n] = v;
        }
        __syncthreads();
    }
}

// Weight and bias gradients, one workgroup per 16 x 16 tile of a layer's
// dW = dz^T h_in (contraction over the batch): blockIdx.x 0 .. 63 layer 2, 64 ..
// 127 layer 1, 128 .. 143 layer 0, 144 .. 151 layer 3.  Wave w of eight takes
// samples 4 (w + 8 q) .. + 3, its sums are added in wave order; the tile of a
// layer's first columns also sums dz itself (the products with ones) into db.
// Samples past the batch read its last one with weight zero, so that a wave's
// loads carry no branch.
constexpr int kMlpGradTiles = 64 + 64 + 16 + 8;

template <int L>
__device__ __forceinline__ void mlp_grad_sums(const float* __restrict__ params, const float* __restrict__ hin,
                                              const float* __restrict__ h2, const float* __restrict__ dy,
                                              const float* __restrict__ dz, int B, int i, int jc, v4f& acc,
                                              v4f& bacc) {
    constexpr int in = L == 0 ? kMlpIn : kMlpWidth, out = L == 3 ? kMlpOut : kMlpWidth;
    const int lane = threadIdx.x & (kWave - 1), lk = lane >> 4;
    const bool iok = i < out, jok = jc < in;
    const int ic = iok ? i : 0, jr = jok ? jc : 0;
    const float wa = L == 2 ? params[mlp_off(3) + ic] : 0.f, wb = L == 2 ? params[mlp_off(3) + kMlpWidth + ic] : 0.f;
    // A[i][k] = dz of sample b + k, B[k][j] = h_in of sample b + k
#pragma unroll 8
    for (int64_t b = 4 * (threadIdx.x / kWave); b < B; b += 4 * (kMlpThreads / kWave)) {
        const bool ok = b + lk < B;
        const int64_t q = ok ? b + lk : B - 1;
        float a;
        if (L == 2)
            a = dz_out(dy[q * kMlpOut], dy[q * kMlpOut + 1], wa, wb, h2[q * kMlpWidth + ic]);
        else
            a = L == 3 ? dy[q * kMlpOut + ic] : dz[q * kMlpWidth + ic];
        a = ok && iok ? a : 0.f;
        const float h = ok && jok ? hin[q * in + jr] : 0.f;
        acc = __builtin_amdgcn_mfma_f32_16x16x4f32(a, h, acc, 0, 0, 0);
        bacc = __builtin_amdgcn_mfma_f32_16x16x4f32(a, 1.f, bacc, 0, 0, 0);
    }
}

__global__ __launch_bounds__(kMlpThreads) void k_mlp_weight_grad(const float* __restrict__ params,
                                                                 const float* __restrict__ x,
                                                                 const float* __restrict__ hidden,
                                                                 const float* __restrict__ dy,
                                                                 const float* __restrict__ dz1,
                                                                 const float* __restrict__ dz0, int B,
                                                                 float* __restrict__ grad) {
    constexpr int kWaves = kMlpThreads / kWave;
    __shared__ float part[kWaves][16 * 16], bpart[kWaves][16];
    const int tid = threadIdx.x, lane = tid & (kWave - 1), w = tid / kWave;
    const int li = lane & 15, lk = lane >> 4;
    const int q = blockIdx.x;
    const int l = q < 64 ? 2 : q < 128 ? 1 : q < 144 ? 0 : 3;
    const int e = l == 2 ? q : l == 1 ? q - 64 : l == 0 ? q - 128 : q - 144;
    const int ncol = l == 0 ? 2 : 8;  // 16-column tiles of the layer's input
    const int i0 = 16 * (e / ncol), j0 = 16 * (e % ncol);
    const int in = l == 0 ? kMlpIn : kMlpWidth, out = l == 3 ? kMlpOut : kMlpWidth;
    const int64_t hs = (int64_t)B * kMlpWidth;
    const float* h2 = hidden + 2 * hs;
    v4f acc = v4f{0.f, 0.f, 0.f, 0.f}, bacc = acc;
    if (l == 2)
        mlp_grad_sums<2>(params, hidden + hs, h2, dy, nullptr, B, i0 + li, j0 + li, acc, bacc);
    else if (l == 1)
        mlp_grad_sums<1>(params, hidden, h2, dy, dz1, B, i0 + li, j0 + li, acc, bacc);
    else if (l == 0)
        mlp_grad_sums<0>(params, x, h2, dy, dz0, B, i0 + li, j0 + li, acc, bacc);
    else
        mlp_grad_sums<3>(params, h2, h2, dy, nullptr, B, i0 + li, j0 + li, acc, bacc);
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        part[w][(4 * lk + r) * 16 + li] = acc[r];
        if (li == 0) bpart[w][4 * lk + r] = bacc[r];
    }
    __syncthreads();
    float* gW = grad + mlp_off(l);
    if (tid < 16 * 16) {
        const int r = tid / 16, c = tid % 16;
        float v = part[0][tid];
#pragma unroll
        for (int u = 1; u < kWaves; ++u) v += part[u][tid];
        if (i0 + r < out && j0 + c < in) gW[(int64_t)(i0 + r) * in + j0 + c] = v;
    } else if (j0 == 0 && tid < 16 * 16 + 16 && i0 + tid - 16 * 16 < out) {
        const int r = tid - 16 * 16;
        float s = bpart[0][r];
#pragma unroll
        for (int u = 1; u < kWaves; ++u) s += bpart[u][r];
        gW[(int64_t)out * in + i0 + r] = s;
    }
}

// Weighted MSE: dY = 2 w_k (Y - T) / B and loss = sum w_k (Y - T)^2 / B
// (one block; the per-thread partial sums are combined in a fixed order).
__global__ __launch_bounds__(kBlock) void k_mse(const float* __restrict__ Y, const float* __restrict__ T,
                                                const float* __restrict__ w, int B, int K, float* __restrict__ loss,
                                                float* __restrict__ dY) {
    __shared__ double lds[kBlock / kWave];
    double s = 0.0;
    const float inv = 1.0f / (float)B;
    for (int e = threadIdx.x; e < B * K; e += kBlock) {
        const int k = e % K;
        const float r = Y[e] - T[e];
        if (dY) dY[e] = 2.f * w[k] * r * inv;
        s += (double)w[k] * (double)r * (double)r;
    }
    s = block_sum<kBlock>(s, lds);
    if (threadIdx.x == 0 && loss) *loss = (float)(s / (double)B);
}

// Adam (bias-corrected): m = b1 m + (1-b1) g, v = b2 v + (1-b2) g^2,
// p -= lr (m c1) / (sqrt(v c2) + eps) with c1 = 1/(1-b1^t), c2 = 1/(1-b2^t).
__global__ __launch_bounds__(kBlock) void k_adam(float* __restrict__ p, const float* __restrict__ g,
                                                 float* __restrict__ m, float* __restrict__ v, int64_t n, float lr,
                                                 float b1, float b2, float eps, float c1, float c2) {
    const int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (i >= n) return;
    const float gi = g[i];
    const float mi = fmaf(b1, m[i], (1.f - b1) * gi);
    const float vi = fmaf(b2, v[i], (1.f - b2) * gi * gi);
    m[i] = mi;
    v[i] = vi;
    p[i] -= lr * (mi * c1) / (sqrtf(vi * c2) + eps);
}

// Standardised predictor input from the first Golub-Kahan scalars:
// x = ((log alpha_1..alpha_p, log beta_2..beta_{p+1}, log kappa, log eps,
// log n, log h) - mean) / std, p = kMlpProbe (one thread).
__global__ void k_mlp_features(const double* __restrict__ alpha, const double* __restrict__ beta, double kappa,
                               double eps, double n, double h, const float* __restrict__ mean,
                               const float* __restrict__ stdv, float* __restrict__ x) {
    if (threadIdx.x != 0 || blockIdx.x != 0) return;
    double raw[kMlpIn];
    for (int j = 0; j < kMlpProbe; ++j) {
        raw[j] = log(alpha[j]);
        raw[kMlpProbe + j] = log(beta[j + 1]);
    }
    raw[2 * kMlpProbe + 0] = log(kappa);
    raw[2 * kMlpProbe + 1] = log(eps);
    raw[2 * kMlpProbe + 2] = log(n);
    raw[2 * kMlpProbe + 3] = log(h);
    for (int i = 0; i < kMlpIn; ++i) x[i] = (float)((raw[i] - (double)mean[i]) / (double)stdv[i]);
}

// ---------------------------------------------------------------------------
// Host launchers
// ---------------------------------------------------------------------------

// hidden: batch x (kMlpLayers - 1) x kMlpWidth, layer-major blocks of
// batch x kMlpWidth (the tanh outputs, kept for the backward pass).  Parameters
// that do not start on 16 bytes are read one at a time.
void launch_mlp_forward(const float* params, const float* x, int B, float* y, float* hidden, hipStream_t s) {
    const unsigned g = (unsigned)((B + kMlpRows - 1) / kMlpRows);
    if (reinterpret_cast<uintptr_t>(params) % 16 == 0)
        k_mlp_forward<true><<<g, kMlpThreads, 0, s>>>(params, x, B, y, hidden);
    else
        k_mlp_forward<false><<<g, kMlpThreads, 0, s>>>(params, x, B, y, hidden);
}

// work: 2 x batch x kMlpWidth floats (dL/dz of layers 1 and 0).
void launch_mlp_backward(const float* params, const float* x, const float* hidden, const float* dy, int B,
                         float* grad, float* work, hipStream_t s) {
    float* dz1 = work;
    float* dz0 = work + (int64_t)B * kMlpWidth;
    k_mlp_data_grad<<<(unsigned)((B + kMlpRows - 1) / kMlpRows), kMlpThreads, 0, s>>>(params, hidden, dy, B, dz1, dz0);
    k_mlp_weight_grad<<<kMlpGradTiles, kMlpThreads, 0, s>>>(params, x, hidden, dy, dz1, dz0, B, grad);
}

void launch_mse(const float* y, const float* t, const float* w, int B, float* loss, float* dy, hipStream_t s) {
    k_mse<<<1, kBlock, 0, s>>>(y, t, w, B, kMlpOut, loss, dy);
}

void launch_adam(float* p, const float* g, float* m, float* v, int64_t n, float lr, float b1, float b2, float eps,
                 int32_t t, hipStream_t s) {
    const float c1 = (float)(1.0 / (1.0 - pow((double)b1, (double)t)));
    const float c2 = (float)(1.0 / (1.0 - pow((double)b2, (double)t)));
    k_adam<<<(unsigned)((n + kBlock - 1) / kBlock), kBlock, 0, s>>>(p, g, m, v, n, lr, b1, b2, eps, c1, c2);
}

void launch_mlp_features(const double* alpha, const double* beta, double kappa, double eps, double n, double h,
                         const float* mean, const float* stdv, float* x, hipStream_t s) {
    k_mlp_features<<<1, 64, 0, s>>>(alpha, beta, kappa, eps, n, h, mean, stdv, x);
}

}  // namespace mqh
