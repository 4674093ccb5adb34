// Cost-model MLP kernels: 16 -> 64 -> 64 -> 2, fp32, ReLU hidden layers.
//
// The model predicts, per instance, [log of sweep time per kernel vector,
// log10 of the survivor density] from the 16 features the packer computes.
// It only orders and sizes work for the persistent scheduler; counts never
// depend on it.
//
// Parameters (WPM_MLP_PARAMS floats): W1[64][16] b1[64] W2[64][64] b2[64]
// W3[2][64] b3[2].  Normalisation (WPM_MLP_NORM floats, not trained):
// mean_x[16] std_x[16] mean_y[2] std_y[2]; inputs are standardised and outputs
// de-standardised inside the kernels.  Loss: mean over samples and outputs of
// the squared error on standardised targets.
//
// Kernels:
//   mlp_forward     a workgroup of 4 waves takes 32 samples: the layers as
//                   16x16x4 fp32 matrix instructions from LDS
//   mlp_tile_grad   the same tile forward, its deltas, and the tile's
//                   parameter gradients and loss (matrix instructions over the
//                   tile's samples), written as one partial sum
//   mlp_reduce      the partial sums of the tiles, in a fixed order
//                   (deterministic, no atomics)
//   mlp_adam        one thread per parameter
//
// All of it is latency-bound: 0.17 GFLOP for 16384 inferences, 30 MFLOP for a
// gradient over 1024 samples.  What counts is that every CU has a tile and that
// no chain is long.  A thread per sample left the deltas of 1024 samples to 4
// workgroups, and a thread per parameter summed the samples one after another
// in 22: a training step (gradient and update, launches included) took 321 us
// for 1024 samples and 1103 us for 4096.  A tile of 32 fills 128 CUs at 4096
// samples: 19 and 20 us, most of it launches; 16 would make more partial sums
// than the work buffer holds.  Prediction of 16384 samples, copies included,
// went from 129 to 106 us.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdint>

#include "internal.h"

namespace wpm {

namespace {
constexpr int IN = 16, H = 64, OUT = 2;
constexpr int OFF_W1 = 0;
constexpr int OFF_B1 = OFF_W1 + H * IN;
constexpr int OFF_W2 = OFF_B1 + H;
constexpr int OFF_B2 = OFF_W2 + H * H;
constexpr int OFF_W3 = OFF_B2 + H;
constexpr int OFF_B3 = OFF_W3 + OUT * H;
constexpr int NPARAM = OFF_B3 + OUT;
constexpr int NNORM = 2 * IN + 2 * OUT;
static_assert(NPARAM == WPM_MLP_PARAMS, "parameter layout");
static_assert(NNORM == WPM_MLP_NORM, "normalisation layout");

// The work buffer (its size is part of the interface): WS floats per sample.
// It holds one partial sum of PS floats per workgroup; a batch of less than 64
// samples, for which it could be too small for two, is one workgroup's.
constexpr int WS = IN + 4 * H + OUT + 1;
constexpr int PS = NPARAM + 2;  // gradients, loss, padding
constexpr int TILE = 32;        // samples of a tile
constexpr int ONE_GROUP = 64;   // smaller batches are one workgroup's
constexpr int MAX_GROUPS = 512; // workgroups of a gradient: larger batches take several tiles each
static_assert(ONE_GROUP * WS >= 2 * PS && TILE * WS >= PS, "partial sums fit the work buffer");

typedef float f4 __attribute__((ext_vector_type(4)));

// LDS rows are padded by one float: the 16 rows that a matrix instruction's
// operand reads start in 16 different banks.
constexpr int LX = IN + 1, LH = H + 1;

struct Weights {
    float w1[H * LX], b1[H], w2[H * LH], b2[H], w3[OUT * H], b3[OUT], norm[NNORM];
};

__device__ __forceinline__ void load_weights(Weights &s, const float *p, const float *norm) {
    const int t = threadIdx.x;
    for (int i = t; i < H * IN; i += 256) s.w1[(i / IN) * LX + i % IN] = p[OFF_W1 + i];
    for (int i = t; i < H * H; i += 256) s.w2[(i / H) * LH + i % H] = p[OFF_W2 + i];
    if (t < H) {
        s.b1[t] = p[OFF_B1 + t];
        s.b2[t] = p[OFF_B2 + t];
    }
    if (t < OUT * H) s.w3[t] = p[OFF_W3 + t];
    if (t < OUT) s.b3[t] = p[OFF_B3 + t];
    if (t < NNORM) s.norm[t] = norm[t];
}

// c += A B over K, for one 16 x 16 tile of a wave: lane l gives a(l % 16, k)
// and b(k, l % 16) for k = l / 16 of each step of 4, and holds the elements
// (4 (l / 16) + r, l % 16) of c.
template <int K, class A, class B>
__device__ __forceinline__ f4 mm(f4 c, A a, B b) {
    const int l16 = threadIdx.x & 15, lk = (threadIdx.x >> 4) & 3;
#pragma unroll
    for (int k = 0; k < K; k += 4) c = __builtin_amdgcn_mfma_f32_16x16x4f32(a(l16, k + lk), b(k + lk, l16), c, 0, 0, 0);
    return c;
}

// Forward pass of samples [b0, b0 + TILE) (rows at and beyond B are zero
// inputs): standardised inputs, activations and the two outputs per sample
// (before de-standardisation).  Wave w computes the hidden units 16 w..16 w + 15.
struct Tile {
    float xn[TILE * LX], a1[TILE * LH], a2[TILE * LH], y[TILE * OUT];
};

__device__ __forceinline__ void forward_tile(const Weights &s, Tile &t, const float *X, int64_t b0, int B) {
    const int tid = threadIdx.x, w16 = (tid >> 6) * 16, l16 = tid & 15, l4 = ((tid >> 4) & 3) * 4;
    for (int i = tid; i < TILE * IN; i += 256) {
        const int r = i / IN, j = i % IN;
        t.xn[r * LX + j] = b0 + r < B ? (X[(b0 + r) * IN + j] - s.norm[j]) / s.norm[IN + j] : 0.0f;
    }
    __syncthreads();
#pragma unroll
    for (int m = 0; m < TILE; m += 16) {
        const float bias = s.b1[w16 + l16];
        const f4 z = mm<IN>(f4{bias, bias, bias, bias}, [&](int i, int k) { return t.xn[(m + i) * LX + k]; },
                            [&](int k, int j) { return s.w1[(w16 + j) * LX + k]; });
#pragma unroll
        for (int r = 0; r < 4; ++r) t.a1[(m + l4 + r) * LH + w16 + l16] = fmaxf(z[r], 0.0f);
    }
    __syncthreads();
#pragma unroll
    for (int m = 0; m < TILE; m += 16) {
        const float bias = s.b2[w16 + l16];
        const f4 z = mm<H>(f4{bias, bias, bias, bias}, [&](int i, int k) { return t.a1[(m + i) * LH + k]; },
                           [&](int k, int j) { return s.w2[(w16 + j) * LH + k]; });
#pragma unroll
        for (int r = 0; r < 4; ++r) t.a2[(m + l4 + r) * LH + w16 + l16] = fmaxf(z[r], 0.0f);
    }
    __syncthreads();
    if (tid < TILE * OUT) {
        const int r = tid / OUT, o = tid % OUT;
        float v = s.b3[o];
#pragma unroll 16
        for (int j = 0; j < H; ++j) v = fmaf(s.w3[o * H + j], t.a2[r * LH + j], v);
        t.y[tid] = v;
    }
}

__global__ __launch_bounds__(256) void mlp_forward(const float *__restrict__ params,
                                                   const float *__restrict__ norm,
                                                   const float *__restrict__ X, int B,
                                                   float *__restrict__ Y) {
    __shared__ Weights s;
    __shared__ Tile t;
    const int64_t b0 = (int64_t)blockIdx.x * TILE;
    load_weights(s, params, norm);
    __syncthreads();
    forward_tile(s, t, X, b0, B);
    const int tid = threadIdx.x;
    if (tid < TILE * OUT && b0 + tid / OUT < B) {  // (each thread wrote the y it reads)
        const int o = tid % OUT;
        Y[b0 * OUT + tid] = t.y[tid] * s.norm[2 * IN + OUT + o] + s.norm[2 * IN + o];
    }
}

// Gradients and loss of a workgroup's tiles: to `part` + PS per workgroup, or,
// when there is only one, gradients and scaled loss to their places.  A thread
// adds to the values that it wrote for the tile before.
__global__ __launch_bounds__(256) void mlp_tile_grad(const float *__restrict__ params,
                                                     const float *__restrict__ norm,
                                                     const float *__restrict__ X,
                                                     const float *__restrict__ T, int B,
                                                     float *__restrict__ part, float *__restrict__ grad,
                                                     float *__restrict__ loss) {
    __shared__ Weights s;
    __shared__ Tile t;
    __shared__ float d1[TILE * LH], d2[TILE * LH], dy[TILE * OUT], se[TILE * OUT];
    const int tid = threadIdx.x, w16 = (tid >> 6) * 16, l16 = tid & 15, l4 = ((tid >> 4) & 3) * 4;
    load_weights(s, params, norm);
    float *g = grad ? grad : part + (int64_t)blockIdx.x * PS;
    float sum = 0.0f;  // of the squared errors (thread 64)
    bool more = false;
    auto put = [&](int i, float v) { g[i] = more ? g[i] + v : v; };
    for (int64_t b0 = (int64_t)blockIdx.x * TILE; b0 < B; b0 += (int64_t)gridDim.x * TILE, more = true) {
    __syncthreads();
    forward_tile(s, t, X, b0, B);
    if (tid < TILE * OUT) {
        const int o = tid % OUT;
        const bool in = b0 + tid / OUT < B;
        const float tn = in ? (T[b0 * OUT + tid] - s.norm[2 * IN + o]) / s.norm[2 * IN + OUT + o] : 0.0f;
        const float e = in ? t.y[tid] - tn : 0.0f;
        const float scale = 2.0f / ((float)B * (float)OUT);
        se[tid] = e * e;
        dy[tid] = scale * e;
    }
    __syncthreads();
    // d2 = (dy W3) where z2 > 0; rows beyond the batch are zero
    for (int i = tid; i < TILE * H; i += 256) {
        const int r = i / H, j = i % H;
        const float v = fmaf(s.w3[H + j], dy[r * OUT + 1], s.w3[j] * dy[r * OUT]);
        d2[r * LH + j] = b0 + r < B && t.a2[r * LH + j] > 0.0f ? v : 0.0f;
    }
    __syncthreads();
    // d1 = (d2 W2) where z1 > 0
#pragma unroll
    for (int m = 0; m < TILE; m += 16) {
        const f4 v = mm<H>(f4{0.0f, 0.0f, 0.0f, 0.0f}, [&](int i, int k) { return d2[(m + i) * LH + k]; },
                           [&](int k, int j) { return s.w2[k * LH + w16 + j]; });
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int row = m + l4 + r, col = w16 + l16;
            d1[row * LH + col] = b0 + row < B && t.a1[row * LH + col] > 0.0f ? v[r] : 0.0f;
        }
    }
    // rows of inputs and activations beyond the batch count for nothing
    if (b0 + TILE > B)
        for (int i = tid; i < TILE * H; i += 256)
            if (b0 + i / H >= B) t.a1[(i / H) * LH + i % H] = t.a2[(i / H) * LH + i % H] = 0.0f;
    __syncthreads();
    // W2: d2^T a1; wave w has the rows 16 w..
#pragma unroll
    for (int n = 0; n < H; n += 16) {
        const f4 v = mm<TILE>(f4{0.0f, 0.0f, 0.0f, 0.0f}, [&](int i, int k) { return d2[k * LH + w16 + i]; },
                              [&](int k, int j) { return t.a1[k * LH + n + j]; });
#pragma unroll
        for (int r = 0; r < 4; ++r) put(OFF_W2 + (w16 + l4 + r) * H + n + l16, v[r]);
    }
    {
        const f4 v = mm<TILE>(f4{0.0f, 0.0f, 0.0f, 0.0f}, [&](int i, int k) { return d1[k * LH + w16 + i]; },
                              [&](int k, int j) { return t.xn[k * LX + j]; });
#pragma unroll
        for (int r = 0; r < 4; ++r) put(OFF_W1 + (w16 + l4 + r) * IN + l16, v[r]);
    }
    // biases, W3 and the loss: sums over the tile's samples
    if (tid < 2 * H) {
        const float *d = tid < H ? d1 + tid : d2 + tid - H;
        float v = 0.0f;
#pragma unroll 8
        for (int r = 0; r < TILE; ++r) v += d[r * LH];
        put(tid < H ? OFF_B1 + tid : OFF_B2 + tid - H, v);
    } else {
        const int o = (tid - 2 * H) / H, j = tid % H;
        float v = 0.0f;
#pragma unroll 8
        for (int r = 0; r < TILE; ++r) v = fmaf(dy[r * OUT + o], t.a2[r * LH + j], v);
        put(OFF_W3 + o * H + j, v);
    }
    if (tid < OUT) {
        float v = 0.0f;
        for (int r = 0; r < TILE; ++r) v += dy[r * OUT + tid];
        put(OFF_B3 + tid, v);
    }
    if (tid == 64)
#pragma unroll 16
        for (int i = 0; i < TILE * OUT; ++i) sum += se[i];
    }
    if (tid == 64) {
        if (!grad)
            g[NPARAM] = sum;
        else if (loss)
            loss[0] = sum / ((float)B * (float)OUT);
    }
}

// Sums of the workgroups' partial sums: 64 values by 8 runs of them a workgroup,
// every sum in the same order each time.
__global__ __launch_bounds__(512) void mlp_reduce(const float *__restrict__ part, int tiles, int B,
                                                  float *__restrict__ grad, float *__restrict__ loss) {
    __shared__ float red[8][64];
    const int c = threadIdx.x & 63, run = threadIdx.x >> 6;
    const int p = blockIdx.x * 64 + c;
    float v = 0.0f;
    if (p <= NPARAM) {
#pragma unroll 8
        for (int i = run; i < tiles; i += 8) v += part[(int64_t)i * PS + p];
    }
    red[run][c] = v;
    __syncthreads();
    if (run == 0 && p <= NPARAM) {
#pragma unroll
        for (int r = 1; r < 8; ++r) v += red[r][c];
        if (p < NPARAM)
            grad[p] = v;
        else if (loss)
            loss[0] = v / ((float)B * (float)OUT);
    }
}

__global__ __launch_bounds__(256) void mlp_adam(float *__restrict__ params,
                                                const float *__restrict__ grad,
                                                float *__restrict__ m, float *__restrict__ v,
                                                float lr, float b1, float b2, float eps,
                                                float bc1, float bc2, float wd) {
    const int p = blockIdx.x * blockDim.x + threadIdx.x;
    if (p >= NPARAM) return;
    const float g = grad[p] + wd * params[p];
    const float mp = b1 * m[p] + (1.0f - b1) * g;
    const float vp = b2 * v[p] + (1.0f - b2) * g * g;
    m[p] = mp;
    v[p] = vp;
    params[p] -= lr * (mp / bc1) / (sqrtf(vp / bc2) + eps);
}

int hip_status(hipError_t e, const char *what) {
    if (e == hipSuccess) return WPM_OK;
    set_hip_error(what, (int)e, hipGetErrorString(e));
    return WPM_EHIP;
}

}  // namespace

int64_t mlp_work_floats(int B) { return (int64_t)B * WS; }

int mlp_forward_launch(const float *params, const float *norm, const float *X, int B, float *Y,
                       void *stream) {
    if (!params || !norm || (B > 0 && (!X || !Y)) || B < 0) return WPM_EINVAL;
    if (B == 0) return WPM_OK;
    hipLaunchKernelGGL(mlp_forward, dim3((unsigned)(((int64_t)B + TILE - 1) / TILE)), dim3(256), 0,
                       (hipStream_t)stream, params, norm, X, B, Y);
    return hip_status(hipGetLastError(), "mlp_forward");
}

int mlp_grad_launch(const float *params, const float *norm, const float *X, const float *T, int B,
                    float *grad, float *work, float *loss, void *stream) {
    if (!params || !norm || !X || !T || !grad || !work || B <= 0) return WPM_EINVAL;
    hipStream_t st = (hipStream_t)stream;
    const bool one = B < ONE_GROUP;
    const int groups = one ? 1 : (int)std::min<int64_t>(MAX_GROUPS, ((int64_t)B + TILE - 1) / TILE);
    hipLaunchKernelGGL(mlp_tile_grad, dim3((unsigned)groups), dim3(256), 0, st, params, norm, X, T, B, work,
                       one ? grad : nullptr, loss);
    const int rc = hip_status(hipGetLastError(), "mlp_tile_grad");
    if (rc || one) return rc;
    hipLaunchKernelGGL(mlp_reduce, dim3((NPARAM + 64) / 64), dim3(512), 0, st, work, groups, B, grad, loss);
    return hip_status(hipGetLastError(), "mlp_reduce");
}

int mlp_adam_launch(float *params, const float *grad, float *m, float *v, int step, float lr,
                    float beta1, float beta2, float eps, float weight_decay, void *stream) {
    if (!params || !grad || !m || !v || step < 1) return WPM_EINVAL;
    const float bc1 = 1.0f - powf(beta1, (float)step);
    const float bc2 = 1.0f - powf(beta2, (float)step);
    hipLaunchKernelGGL(mlp_adam, dim3((NPARAM + 255) / 256), dim3(256), 0, (hipStream_t)stream,
                       params, grad, m, v, lr, beta1, beta2, eps, bc1, bc2, weight_decay);
    return hip_status(hipGetLastError(), "mlp_adam");
}

}  // namespace wpm
