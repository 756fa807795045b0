// pt_mlp.hip -- FP32 training and inference kernels of the ladder network.
//
// The network maps 32 instance features to 64 outputs: 32 -> 128 -> 128 -> 64 with ReLU
// after the two hidden layers.  Parameters, flat FP32 in this order:
//   W1[128][32], b1[128], W2[128][128], b2[128], W3[64][128], b3[64]   (28,992 floats)
// Two training losses (targets q[batch][64]):
//   PT_MLP_LOSS_SOFTMAX:  -sum_j q_j log softmax(z)_j                 (q rows sum to 1)
//   PT_MLP_LOSS_SIGMOID:  -sum_j [q_j log s(z_j) + (1-q_j) log(1-s(z_j))], s = logistic
// both averaged over the batch; either has gradient (p - q)/B in the logits.
//
// Every dense product runs on the matrix cores with v_mfma_f32_16x16x4f32.  The network is
// small enough that launches and dependent trips to memory are its whole cost, so a call is
// one launch (forward) or two (loss and gradients):
//   mlp_rows    16 rows of the batch through all layers by one workgroup of eight waves, one
//               16-column tile each; activations pass through LDS, and each wave's slices of
//               every weight matrix are loaded before the first product.  With GRAD also the
//               loss and the gradients of the three layers' outputs.
//   mlp_grads   weight gradients, one 16x16 tile per workgroup, the batch split over its
//               waves; bias gradients ride along in the tiles of the first columns.
// Measured on MI355X with the binding's Python: loss, gradients and Adam at batch 256 261 -> 46 us
// (thirteen launches and column sums by one thread per column before), a forward pass of 512
// rows 20.2 -> 9.7 us (three launches before, and now mostly Python).
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <cmath>
#include <string>

#include "../../include/ptqmc.h"
#include "pt_internal.h"

namespace {

// PT_OK, or PT_EHIP with the HIP error recorded as the last error
int launched(hipError_t e, const char *what)
{
    if (e == hipSuccess) return PT_OK;
    return ptq::report_error(PT_EHIP, (std::string(what) + ": " + hipGetErrorString(e)).c_str());
}

constexpr int kIn = 32, kH = 128, kOut = 64;
constexpr int kW1 = 0, kB1 = kW1 + kH * kIn, kW2 = kB1 + kH, kB2 = kW2 + kH * kH,
              kW3 = kB2 + kH, kB3 = kW3 + kOut * kH, kParams = kB3 + kOut;

typedef float v4f __attribute__((ext_vector_type(4)));
// four floats at any float's alignment (the caller's pointers promise no more)
typedef float v4u __attribute__((ext_vector_type(4), aligned(4)));

constexpr int kRows = 16;        // rows of the batch per workgroup
constexpr int kRowThreads = 512; // eight waves: one 16-column tile of a hidden layer each
// LDS rows are padded by four floats, so that the sixteen rows a wave reads 16 bytes of at a
// time start on different banks
constexpr int kInL = kIn + 4, kHL = kH + 4, kOutL = kOut + 4;

// Product of an LDS tile a[16][lda] with the columns whose weights the lanes hold: in step
// (c, s) lane quarter kq takes k = 16 c + 4 kq + s on both sides.
template <int K>
__device__ __forceinline__ v4f tile_mul(const float *a, int lda, const float (&w)[K / 4], int r16, int kq)
{
    v4f acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int c = 0; c < K / 16; ++c) {
        const v4f v = *reinterpret_cast<const v4f *>(a + r16 * lda + 16 * c + 4 * kq);
#pragma unroll
        for (int s = 0; s < 4; ++s) acc = __builtin_amdgcn_mfma_f32_16x16x4f32(v[s], w[4 * c + s], acc, 0, 0, 0);
    }
    return acc;
}

// A lane's weights of column n = row n of W[.][K] (y = x W^T), or column n of W[K][ld] (dx = dy W).
template <int K>
__device__ __forceinline__ void load_rows(const float *W, int n, int kq, float (&w)[K / 4])
{
#pragma unroll
    for (int c = 0; c < K / 16; ++c) {
        const v4u v = *reinterpret_cast<const v4u *>(W + n * K + 16 * c + 4 * kq);
#pragma unroll
        for (int s = 0; s < 4; ++s) w[4 * c + s] = v[s];
    }
}
template <int K>
__device__ __forceinline__ void load_cols(const float *W, int ld, int n, int kq, float (&w)[K / 4])
{
#pragma unroll
    for (int c = 0; c < K / 16; ++c)
#pragma unroll
        for (int s = 0; s < 4; ++s) w[4 * c + s] = W[(16 * c + 4 * kq + s) * ld + n];
}

struct Acts {
    float *h1, *h2, *dz3, *dz2, *dz1, *loss;
};

// Loss of one row and its gradient in logit j (lane j): softmax cross entropy against soft
// targets, or per-output logistic cross entropy (log(1 + e^{-|v|}) + max(v, 0) - q v).
__device__ __forceinline__ void row_loss(int kind, float v, float tq, float &d, float &l)
{
    if (kind == PT_MLP_LOSS_SOFTMAX) {
        float mx = v;
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) mx = fmaxf(mx, __shfl_xor(mx, off, 64));
        const float ex = __expf(v - mx);
        float sum = ex;
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) sum += __shfl_xor(sum, off, 64);
        d = ex / sum - tq;
        l = (tq > 0.f) ? -tq * (v - mx - __logf(sum)) : 0.f;
    } else {
        d = 1.f / (1.f + __expf(-v)) - tq;
        l = __logf(1.f + __expf(-fabsf(v))) + fmaxf(v, 0.f) - tq * v;
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) l += __shfl_xor(l, off, 64);
}

// Logits of a call without a workspace whose logits overlap its inputs (forward).
__device__ float aside[(size_t)PT_MLP_STATIC_MAX_BATCH * kOut];

__global__ void copy_aside_kernel(float *logits, int n)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) logits[i] = aside[i];
}

// logits: null for `aside`.
template <bool GRAD>
__global__ void __launch_bounds__(kRowThreads) mlp_rows_kernel(const float *P, const float *x, const float *q,
                                                               float *logits, Acts g, int B, int kind)
{
    __shared__ __align__(16) float xs[kRows * kInL], h1s[kRows * kHL], h2s[kRows * kHL], zs[kRows * kOutL],
        ds[kRows * kHL];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int r16 = lane & 15, kq = lane >> 4;
    const int m0 = blockIdx.x * kRows;
    const int col = 16 * wave + r16;  // the lane's column of a hidden layer
    // every weight this wave will need, in flight at once
    float w1[kIn / 4], w2[kH / 4], w3[kH / 4], w3t[kOut / 4], w2t[kH / 4];
    load_rows<kIn>(P + kW1, col, kq, w1);
    load_rows<kH>(P + kW2, col, kq, w2);
    load_rows<kH>(P + kW3, 16 * (wave & 3) + r16, kq, w3);
    if constexpr (GRAD) {
        load_cols<kOut>(P + kW3, kH, col, kq, w3t);
        load_cols<kH>(P + kW2, kH, col, kq, w2t);
    }
    const float b1 = P[kB1 + col], b2 = P[kB2 + col], b3 = P[kB3 + 16 * (wave & 3) + r16];
    {
        const int row = threadIdx.x / kIn, k = threadIdx.x % kIn;  // 512 values, one each
        xs[row * kInL + k] = m0 + row < B ? x[(int64_t)(m0 + row) * kIn + k] : 0.f;
    }
    __syncthreads();
    auto hidden = [&](const v4f &acc, float bias, float *out, float *save) {
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int row = 4 * kq + e;
            float v = acc[e] + bias;
            v = v > 0.f ? v : 0.f;
            out[row * kHL + col] = v;
            if (GRAD && m0 + row < B) save[(int64_t)(m0 + row) * kH + col] = v;
        }
    };
    hidden(tile_mul<kIn>(xs, kInL, w1, r16, kq), b1, h1s, g.h1);
    __syncthreads();
    hidden(tile_mul<kH>(h1s, kHL, w2, r16, kq), b2, h2s, g.h2);
    __syncthreads();
    if (wave < kOut / 16) {
        const v4f acc = tile_mul<kH>(h2s, kHL, w3, r16, kq);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int row = 4 * kq + e;
            const float v = acc[e] + b3;
            if constexpr (GRAD) {
                zs[row * kOutL + col] = v;
            } else {
                if (m0 + row < B) (logits ? logits : aside)[(int64_t)(m0 + row) * kOut + col] = v;
            }
        }
    }
    if constexpr (GRAD) {
        __syncthreads();
        // two rows per wave, one logit per lane
#pragma unroll
        for (int e = 0; e < 2; ++e) {
            const int row = 2 * wave + e;
            const bool in = m0 + row < B;
            float d, l;
            row_loss(kind, zs[row * kOutL + lane], in ? q[(int64_t)(m0 + row) * kOut + lane] : 0.f, d, l);
            d = in ? d / (float)B : 0.f;
            zs[row * kOutL + lane] = d;
            if (in) {
                g.dz3[(int64_t)(m0 + row) * kOut + lane] = d;
                if (lane == 0) g.loss[m0 + row] = l;
            }
        }
        __syncthreads();
        // dz of a hidden layer: (dy W) where the stored activation is positive
        auto masked = [&](const v4f &acc, const float *h, float *out, float *save) {
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int row = 4 * kq + e;
                const float v = h[row * kHL + col] > 0.f ? acc[e] : 0.f;
                if (out) out[row * kHL + col] = v;
                if (m0 + row < B) save[(int64_t)(m0 + row) * kH + col] = v;
            }
        };
        masked(tile_mul<kOut>(zs, kOutL, w3t, r16, kq), h2s, ds, g.dz2);
        __syncthreads();
        masked(tile_mul<kH>(ds, kHL, w2t, r16, kq), h1s, nullptr, g.dz1);
    }
}

// Weight gradients dW[o][j] = sum_b dz[b][o] a[b][j] in tiles of 16 x 16: 4 x 8 of layer 3,
// 8 x 8 of layer 2, 8 x 2 of layer 1; db[o] = sum_b dz[b][o] with each layer's first column
// of tiles.  The waves of a workgroup take consecutive runs of the batch (64 rows each up to
// 16 waves), summed through LDS in wave order.  One more workgroup sums the rows' losses.
constexpr int kGradTiles = 32 + 64 + 16;
constexpr int kGradWaves = 16;

__global__ void __launch_bounds__(64 * kGradWaves) mlp_grads_kernel(Acts g, const float *x, float *G, float *loss, int B)
{
    __shared__ float red[kGradWaves][16 * 16], bred[kGradWaves][16];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, waves = blockDim.x >> 6;
    const int t = blockIdx.x;
    if (t == kGradTiles) {
        float s = 0.f;
        for (int b = threadIdx.x; b < B; b += blockDim.x) s += g.loss[b];
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) s += __shfl_xor(s, off, 64);
        if (lane == 0) bred[wave][0] = s;
        __syncthreads();
        if (threadIdx.x == 0) {
            s = 0.f;
            for (int w = 0; w < waves; ++w) s += bred[w][0];
            loss[0] = s;
        }
        return;
    }
    const int r16 = lane & 15, kq = lane >> 4;
    const float *dz, *in;
    float *dW, *db;
    int ldz, ldi, o0, j0;
    if (t < 32) {
        dz = g.dz3, ldz = kOut, in = g.h2, ldi = kH, dW = G + kW3, db = G + kB3, o0 = 16 * (t / 8), j0 = 16 * (t % 8);
    } else if (t < 96) {
        dz = g.dz2, ldz = kH, in = g.h1, ldi = kH, dW = G + kW2, db = G + kB2, o0 = 16 * ((t - 32) / 8), j0 = 16 * ((t - 32) % 8);
    } else {
        dz = g.dz1, ldz = kH, in = x, ldi = kIn, dW = G + kW1, db = G + kB1, o0 = 16 * ((t - 96) / 2), j0 = 16 * ((t - 96) % 2);
    }
    const int per = ((B + waves - 1) / waves + 3) & ~3;  // rows of a wave
    const int begin = wave * per, end = min(B, begin + per);
    v4f acc = {0.f, 0.f, 0.f, 0.f};
    float bias = 0.f;
#pragma unroll 8
    for (int k0 = begin; k0 < end; k0 += 4) {
        // rows past the run's end are read at the last one and count as 0
        const int k = k0 + kq, kk = min(k, B - 1);
        float a = dz[(int64_t)kk * ldz + o0 + r16], b = in[(int64_t)kk * ldi + j0 + r16];
        a = k < end ? a : 0.f;
        b = k < end ? b : 0.f;
        bias += a;
        acc = __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, acc, 0, 0, 0);
    }
    // D[i][j] sits in lane j + 16 * (i / 4), element i % 4
#pragma unroll
    for (int e = 0; e < 4; ++e) red[wave][(4 * kq + e) * 16 + r16] = acc[e];
    bias += __shfl_xor(bias, 16, 64);
    bias += __shfl_xor(bias, 32, 64);
    if (lane < 16) bred[wave][lane] = bias;
    __syncthreads();
    for (int i = threadIdx.x; i < 256; i += blockDim.x) {
        float s = 0.f;
        for (int w = 0; w < waves; ++w) s += red[w][i];
        dW[(o0 + i / 16) * ldi + j0 + i % 16] = s;
    }
    if (j0 == 0 && threadIdx.x < 16) {
        float s = 0.f;
        for (int w = 0; w < waves; ++w) s += bred[w][threadIdx.x];
        db[o0 + threadIdx.x] = s;
    }
}

// Adam (Kingma & Ba): m = b1 m + (1-b1) g; v = b2 v + (1-b2) g^2;
// p -= lr * (m / (1 - b1^t)) / (sqrt(v / (1 - b2^t)) + eps).
__global__ void adam_kernel(float *p, const float *g, float *m, float *v, int n, float lr,
                            float b1, float b2, float eps, float c1, float c2)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const float gi = g[i];
    const float mi = b1 * m[i] + (1.f - b1) * gi;
    const float vi = b2 * v[i] + (1.f - b2) * gi * gi;
    m[i] = mi;
    v[i] = vi;
    p[i] -= lr * (mi / c1) / (sqrtf(vi / c2) + eps);
}

// The part of a workspace each intermediate of B rows takes (pt_mlp_workspace_bytes).
Acts carve(void *ws, int B)
{
    Acts a;
    a.h1 = (float *)ws;
    a.h2 = a.h1 + (size_t)B * kH;
    a.dz3 = a.h2 + (size_t)B * kH;
    a.dz2 = a.dz3 + (size_t)B * kOut;
    a.dz1 = a.dz2 + (size_t)B * kH;
    a.loss = a.dz1 + (size_t)B * kH;
    return a;
}

bool overlap(const float *a, size_t na, const float *b, size_t nb)
{
    const uintptr_t x = (uintptr_t)a, y = (uintptr_t)b;
    return x < y + 4 * nb && y < x + 4 * na;
}

// A workgroup writes its logits while others may still read x and the parameters.  Where the
// logits overlap those they go to the workspace (or, without one, `aside`) first.
hipError_t forward(hipStream_t s, const float *P, const float *x, float *out, int B, float *ws)
{
    const size_t n = (size_t)B * kOut;
    const bool over = overlap(out, n, x, (size_t)B * kIn) || overlap(out, n, P, kParams);
    hipLaunchKernelGGL(mlp_rows_kernel<false>, dim3((B + kRows - 1) / kRows), dim3(kRowThreads), 0, s, P, x,
                       (const float *)nullptr, over ? ws : out, Acts{}, B, 0);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess || !over) return e;
    if (ws) return hipMemcpyAsync(out, ws, n * sizeof(float), hipMemcpyDeviceToDevice, s);
    hipLaunchKernelGGL(copy_aside_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, out, (int)n);
    return hipGetLastError();
}

}  // namespace

extern "C" {

int32_t pt_mlp_param_count(void) { return kParams; }

size_t pt_mlp_workspace_bytes(int32_t batch)
{
    if (batch < 1) return 0;
    return sizeof(float) * ((size_t)batch * (kH + kH + kOut + kOut + kH + kH) + (size_t)batch);
}

int pt_mlp_forward(const float *params, const float *x, float *logits, int32_t batch,
                   void *workspace, void *stream)
{
    if (!params || !x || !logits || !workspace)
        return ptq::report_error(PT_EINVAL, "pt_mlp_forward: null pointer");
    if (batch < 1) return ptq::report_error(PT_EINVAL, "pt_mlp_forward: batch < 1");
    return launched(forward((hipStream_t)stream, params, x, logits, batch, (float *)workspace), "pt_mlp_forward");
}

int pt_mlp_forward_static(const float *params, const float *x, float *logits, int32_t batch,
                          void *stream)
{
    if (!params || !x || !logits)
        return ptq::report_error(PT_EINVAL, "pt_mlp_forward_static: null pointer");
    if (batch < 1) return ptq::report_error(PT_EINVAL, "pt_mlp_forward_static: batch < 1");
    if (batch > PT_MLP_STATIC_MAX_BATCH)
        return ptq::report_error(PT_EINVAL, ("pt_mlp_forward_static: batch " + std::to_string(batch) +
                                             " exceeds PT_MLP_STATIC_MAX_BATCH (" +
                                             std::to_string(PT_MLP_STATIC_MAX_BATCH) + ")").c_str());
    return launched(forward((hipStream_t)stream, params, x, logits, batch, nullptr), "pt_mlp_forward_static");
}

int pt_mlp_loss_grad(const float *params, const float *x, const float *target, int32_t batch,
                     int32_t loss_kind, float *grads, float *loss, void *workspace, void *stream)
{
    if (!params || !x || !target || !grads || !loss || !workspace)
        return ptq::report_error(PT_EINVAL, "pt_mlp_loss_grad: null pointer");
    if (batch < 1) return ptq::report_error(PT_EINVAL, "pt_mlp_loss_grad: batch < 1");
    if (loss_kind != PT_MLP_LOSS_SOFTMAX && loss_kind != PT_MLP_LOSS_SIGMOID)
        return ptq::report_error(PT_EINVAL, "pt_mlp_loss_grad: unknown loss kind");
    hipStream_t s = (hipStream_t)stream;
    const Acts a = carve(workspace, batch);
    const int B = batch;
    hipLaunchKernelGGL(mlp_rows_kernel<true>, dim3((B + kRows - 1) / kRows), dim3(kRowThreads), 0, s, params, x,
                       target, (float *)nullptr, a, B, (int)loss_kind);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return launched(e, "pt_mlp_loss_grad");
    const int waves = B < 64 ? 1 : B >= 64 * kGradWaves ? kGradWaves : (B + 63) / 64;
    hipLaunchKernelGGL(mlp_grads_kernel, dim3(kGradTiles + 1), dim3(64 * waves), 0, s, a, x, grads, loss, B);
    return launched(hipGetLastError(), "pt_mlp_loss_grad");
}

int pt_mlp_adam(float *params, const float *grads, float *m, float *v, int32_t n, float lr,
                float beta1, float beta2, float eps, int32_t step, void *stream)
{
    if (!params || !grads || !m || !v) return ptq::report_error(PT_EINVAL, "pt_mlp_adam: null pointer");
    if (n < 1 || step < 1) return ptq::report_error(PT_EINVAL, "pt_mlp_adam: n < 1 or step < 1");
    // bias corrections 1 - beta^step
    const float c1 = (float)(1.0 - std::pow((double)beta1, (double)step));
    const float c2 = (float)(1.0 - std::pow((double)beta2, (double)step));
    hipLaunchKernelGGL(adam_kernel, dim3((n + 255) / 256), dim3(256), 0, (hipStream_t)stream,
                       params, grads, m, v, n, lr, beta1, beta2, eps, c1, c2);
    return launched(hipGetLastError(), "pt_mlp_adam");
}

}  // extern "C"
