// FP32 kernels of the learned cost model (3 hidden layers of width 64,
// ReLU, scalar output) for gfx950: forward, backward, gradient reduction and
// Adam.  The network predicts the log run time of a loop nest under a launch
// configuration from a standardised feature vector.
//
//   h1 = relu(W1 x + b1), h2 = relu(W2 h1 + b2), h3 = relu(W3 h2 + b3)
//   yhat = w4 . h3 + b4 ;  L = mean_b (yhat_b - y_b)^2 ;  relu'(0) = 0
//
// Parameter vector layout (floats): W1 [64 x F] | b1 [64] | W2 [64 x 64] |
// b2 | W3 [64 x 64] | b3 | w4 [64] | b4 [1].
//
// What bounds it: a minibatch of 256 samples is 14 MFLOP, far below what the
// chip does in the time of one launch, and the steps of a fit depend on each
// other, so a step costs its launches and the latency of its longest chain.
// One lane per sample (9,000 dependent multiply-adds a lane, on two compute
// units) took 143 us forward, 98 us for the deltas, 69 us for the gradients
// and two more launches of 5 us.  Here a workgroup takes 16 samples through
// the whole network on the FP32 matrix cores, so a minibatch spreads over 16
// compute units, its longest chain is about 60 matrix instructions, and a
// step is two launches: gradient partials (8.9 us) and their sum with Adam
// (3.0 us).  An epoch of 2000 samples: 2667 us before, 218 us now; the
// predictions of 20,000 samples 205 and 80 us, of 30 samples 165 and 35 us.
#include "k_common.h"
#include "kernels.h"
#include "mlp_walk.h"

namespace jk {

namespace {

constexpr int H = kMlpHidden;

struct Off {
    int W1, b1, W2, b2, W3, b3, w4, b4, P;
};

__host__ __device__ inline Off offsets(int F) {
    Off o;
    o.W1 = 0;
    o.b1 = o.W1 + H * F;
    o.W2 = o.b1 + H;
    o.b2 = o.W2 + H * H;
    o.W3 = o.b2 + H;
    o.b3 = o.W3 + H * H;
    o.w4 = o.b3 + H;
    o.b4 = o.w4 + H;
    o.P = o.b4 + 1;
    return o;
}

typedef float f4 __attribute__((ext_vector_type(4)));
typedef float f4u __attribute__((ext_vector_type(4), aligned(4)));  // in memory: any float address

constexpr int kTile = kMlpTile;        // samples of a workgroup's tile
constexpr int kThreads = kMlpThreads;  // 4 waves, wave w computing outputs 16w .. 16w+15 of a layer
// LDS row strides: 4 floats past a multiple of 16, so the 16 rows that a
// quarter of a wave reads 16 bytes of lie in different banks
constexpr int SX = kMlpMaxFeatures + 4;
constexpr int SH = H + 4;
static_assert(H == 64 && kMlpMaxFeatures == 16, "the tile layout is written for 64 wide layers, 16 features");

// acc + (16 x 16 product over 16 k's): lane l = 16q + c holds a[t] =
// A[c][k(q, t)] and b[t] = B[k(q, t)][c]; any assignment k(q, t) serves, as
// long as both sides use the same, so each lane takes 4 neighbouring k's
// (4q .. 4q+3) and its operands are 16-byte reads.  acc[r] is element
// [4q + r][c].
__device__ __forceinline__ f4 mma16(f4 a, f4 b, f4 acc) {
#pragma unroll
    for (int t = 0; t < 4; ++t) acc = __builtin_amdgcn_mfma_f32_16x16x4f32(a[t], b[t], acc, 0, 0, 0);
    return acc;
}

// One layer for the tile: rows of `in` (LDS, stride SH) times this wave's 16
// rows of weights (operands in registers).
__device__ __forceinline__ f4 layer(const float *in, int c, int q, const f4 (&w)[4], f4 acc) {
#pragma unroll
    for (int m = 0; m < 4; ++m) acc = mma16(*reinterpret_cast<const f4 *>(&in[c * SH + 16 * m + 4 * q]), w[m], acc);
    return acc;
}

// ReLU of a layer's sums; rows past the last sample are zeroed, so nothing
// of them reaches a gradient.
__device__ __forceinline__ f4 relu(f4 z, int valid) {
    f4 h;
#pragma unroll
    for (int r = 0; r < 4; ++r) h[r] = (r < valid && z[r] > 0.f) ? z[r] : 0.f;
    return h;
}

__device__ __forceinline__ void put(float *to, int q, int o, f4 v) {
#pragma unroll
    for (int r = 0; r < 4; ++r) to[(4 * q + r) * SH + o] = v[r];
}

// sum over the four 16-lane groups of a wave, fixed order
__device__ __forceinline__ float over_q(float v) {
    v += __shfl_xor(v, 16, kWave);
    v += __shfl_xor(v, 32, kWave);
    return v;
}

// The forward pass of samples [0, n) (idx, optional, maps sample b to row
// idx[b] of X), and for TRAIN the backward pass: workgroup g walks the
// 16-sample tiles g, g + grid, ... keeping its gradient sums in registers,
// and writes them to part[g * P ..] (parameter order) and the sum of its
// squared errors to loss[g].  Every sum is in a fixed order.
//   deltas: g = 2 (yhat - y)/n; d3 = g w4 [h3>0]; d2 = W3^T d3 [h2>0];
//   d1 = W2^T d2 [h1>0]
// The accumulator layout of a layer's output (sample 4q + r, output 16w + c)
// is the operand layout of d^T in the gradient products d^T h, so those take
// their left operand straight from registers.
template <bool TRAIN>
__global__ void __launch_bounds__(kThreads)
mlp_tile_kernel(const float *__restrict__ params, const float *__restrict__ mu, const float *__restrict__ sd,
                const float *__restrict__ X, const int *__restrict__ idx, const float *__restrict__ y, int n, int F,
                float *__restrict__ yhat, float *__restrict__ part, double *__restrict__ loss) {
    __shared__ __align__(16) float xs[kTile * SX], h1[kTile * SH], h2[kTile * SH], d[kTile * SH];
    __shared__ float ysum[4][kTile], gs[kTile];
    const Off off = offsets(F);
    const int tid = threadIdx.x, lane = tid & (kWave - 1), w = tid / kWave;
    const int c = lane & 15, q = lane >> 4, o = 16 * w + c;

    // this lane's operands of every layer, kept over all tiles
    f4 w1, w2[4], w3[4], w2t[4], w3t[4];
#pragma unroll
    for (int t = 0; t < 4; ++t) w1[t] = 4 * q + t < F ? params[off.W1 + o * F + 4 * q + t] : 0.f;
#pragma unroll
    for (int m = 0; m < 4; ++m) {
        w2[m] = *reinterpret_cast<const f4u *>(&params[off.W2 + o * H + 16 * m + 4 * q]);
        w3[m] = *reinterpret_cast<const f4u *>(&params[off.W3 + o * H + 16 * m + 4 * q]);
        if (TRAIN) {
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                w2t[m][t] = params[off.W2 + (16 * m + 4 * q + t) * H + o];
                w3t[m][t] = params[off.W3 + (16 * m + 4 * q + t) * H + o];
            }
        }
    }
    const float b1 = params[off.b1 + o], b2 = params[off.b2 + o], b3 = params[off.b3 + o], w4 = params[off.w4 + o];
    const float b4 = params[off.b4];
    const f4 zero = {0.f, 0.f, 0.f, 0.f};
    f4 gw1 = zero, gw2[4] = {zero, zero, zero, zero}, gw3[4] = {zero, zero, zero, zero};
    float gb1 = 0.f, gb2 = 0.f, gb3 = 0.f, gw4 = 0.f, gb4 = 0.f;
    double sq = 0.0;

    const int fs = tid >> 4, ff = tid & 15;  // the sample and feature this thread stages
    const float fmu = ff < F ? mu[ff] : 0.f, fsd = ff < F ? sd[ff] : 1.f;
    for (int64_t base = mlp_first(blockIdx.x); base < n; base = mlp_next(base, gridDim.x)) {
        const int64_t b = base + fs;
        float xv = 0.f;
        if (b < n && ff < F) xv = (X[(idx ? idx[b] : b) * F + ff] - fmu) / fsd;
        xs[fs * SX + ff] = xv;
        __syncthreads();
        const int valid = (int)(n - base < kTile ? n - base : kTile) - 4 * q;  // rows r < valid of this lane's four are samples
        const f4 h1r = relu(mma16(*reinterpret_cast<const f4 *>(&xs[c * SX + 4 * q]), w1, f4{b1, b1, b1, b1}), valid);
        put(h1, q, o, h1r);
        __syncthreads();
        const f4 h2r = relu(layer(h1, c, q, w2, f4{b2, b2, b2, b2}), valid);
        put(h2, q, o, h2r);
        __syncthreads();
        const f4 h3r = relu(layer(h2, c, q, w3, f4{b3, b3, b3, b3}), valid);
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            float p = w4 * h3r[r];
#pragma unroll
            for (int m = 1; m < 16; m <<= 1) p += __shfl_xor(p, m, kWave);
            if (c == 0) ysum[w][4 * q + r] = p;
        }
        __syncthreads();
        if (tid < kTile) {
            const float yh = b4 + ((ysum[0][tid] + ysum[1][tid]) + (ysum[2][tid] + ysum[3][tid]));
            const bool in = base + tid < n;
            if (!TRAIN) {
                if (in) yhat[base + tid] = yh;
            } else {
                const float e = in ? yh - y[idx ? idx[base + tid] : base + tid] : 0.f;
                const float g = 2.f * e / (float)n;
                sq += (double)(e * e);
                gs[tid] = g;
                gb4 += g;
            }
        }
        if (!TRAIN) continue;  // the next tile's first barrier orders the reads of ysum before its next writes
        __syncthreads();
        f4 dr;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const float g = gs[4 * q + r];
            dr[r] = h3r[r] > 0.f ? g * w4 : 0.f;
            gw4 += g * h3r[r];
            gb3 += dr[r];
        }
        put(d, q, o, dr);
#pragma unroll
        for (int j = 0; j < 4; ++j)
#pragma unroll
            for (int r = 0; r < 4; ++r)
                gw3[j] = __builtin_amdgcn_mfma_f32_16x16x4f32(dr[r], h2[(4 * q + r) * SH + 16 * j + c], gw3[j], 0, 0, 0);
        __syncthreads();
        f4 z = layer(d, c, q, w3t, zero);
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            dr[r] = h2r[r] > 0.f ? z[r] : 0.f;
            gb2 += dr[r];
        }
        __syncthreads();  // every wave has read d3
        put(d, q, o, dr);
#pragma unroll
        for (int j = 0; j < 4; ++j)
#pragma unroll
            for (int r = 0; r < 4; ++r)
                gw2[j] = __builtin_amdgcn_mfma_f32_16x16x4f32(dr[r], h1[(4 * q + r) * SH + 16 * j + c], gw2[j], 0, 0, 0);
        __syncthreads();
        z = layer(d, c, q, w2t, zero);
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            dr[r] = h1r[r] > 0.f ? z[r] : 0.f;
            gb1 += dr[r];
        }
#pragma unroll
        for (int r = 0; r < 4; ++r)
            gw1 = __builtin_amdgcn_mfma_f32_16x16x4f32(dr[r], xs[(4 * q + r) * SX + c], gw1, 0, 0, 0);
        __syncthreads();  // the next tile rewrites xs
    }
    if (!TRAIN) return;
    float *g = part + (int64_t)blockIdx.x * off.P;
    const int i0 = 16 * w + 4 * q;  // gradient rows i0 .. i0+3, columns 16j + c
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        if (c < F) g[off.W1 + (i0 + r) * F + c] = gw1[r];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            g[off.W2 + (i0 + r) * H + 16 * j + c] = gw2[j][r];
            g[off.W3 + (i0 + r) * H + 16 * j + c] = gw3[j][r];
        }
    }
    gb1 = over_q(gb1);
    gb2 = over_q(gb2);
    gb3 = over_q(gb3);
    gw4 = over_q(gw4);
    if (q == 0) {
        g[off.b1 + o] = gb1;
        g[off.b2 + o] = gb2;
        g[off.b3 + o] = gb3;
        g[off.w4 + o] = gw4;
    }
    if (tid < kTile) {
#pragma unroll
        for (int m = 1; m < kTile; m <<= 1) {
            gb4 += __shfl_xor(gb4, m, kTile);
            sq += __shfl_xor(sq, m, kTile);
        }
        if (tid == 0) {
            g[off.b4] = gb4;
            loss[blockIdx.x] = sq;
        }
    }
}

struct Adam {
    float *p, *m, *v;  // parameters and moments (p null: gradient only)
    float lr, c1, c2;  // step size and the two bias corrections 1 - beta^t
};

__device__ __forceinline__ void adam(const Adam &A, int k, float g) {
    constexpr float beta1 = 0.9f, beta2 = 0.999f, eps = 1e-8f;
    const float mk = beta1 * A.m[k] + (1.f - beta1) * g;
    const float vk = beta2 * A.v[k] + (1.f - beta2) * g * g;
    A.m[k] = mk;
    A.v[k] = vk;
    A.p[k] = A.p[k] - A.lr * (mk / A.c1) / (sqrtf(vk / A.c2) + eps);
}

// One lane per parameter: its gradient summed over the workgroups' partials
// in order (all loads independent), then its Adam step; workgroup 0's first
// wave also turns the squared errors into the mean loss.
__global__ void __launch_bounds__(kThreads)
mlp_reduce_kernel(const float *__restrict__ part, const double *__restrict__ loss, int groups, int P, int n, Adam A,
                  float *__restrict__ grad, float *__restrict__ loss_out) {
    const int k = blockIdx.x * kThreads + threadIdx.x;
    if (blockIdx.x == 0 && threadIdx.x < kWave) {
        const double t = wave_sum((int)threadIdx.x < groups ? loss[threadIdx.x] : 0.0);
        if (threadIdx.x == 0) *loss_out = (float)(t / (double)n);
    }
    if (k >= P) return;
    float s = 0.f;
    for (int g = 0; g < groups; g += 16) {
        float v[16];
#pragma unroll
        for (int u = 0; u < 16; ++u) v[u] = g + u < groups ? part[(int64_t)(g + u) * P + k] : 0.f;
#pragma unroll
        for (int u = 0; u < 16; ++u) s += v[u];
    }
    grad[k] = s;
    if (A.p) adam(A, k, s);
}

// Adam with bias correction on a gradient computed earlier.
__global__ void __launch_bounds__(kThreads) mlp_adam_kernel(Adam A, const float *__restrict__ grad, int P) {
    const int k = blockIdx.x * kThreads + threadIdx.x;
    if (k < P) adam(A, k, grad[k]);
}

Adam adam_args(const MlpBufs &B, int t, float lr) {
    return {B.params, B.m, B.v, lr, (float)(1.0 - pow((double)0.9f, t)), (float)(1.0 - pow((double)0.999f, t))};
}

unsigned param_blocks(int P) { return (unsigned)((P + kThreads - 1) / kThreads); }

}  // namespace

static_assert(kMlpGroups <= kWave, "one wave sums the groups' squared errors");

int mlp_nparams(int F) { return offsets(F).P; }

hipError_t mlp_forward(const MlpBufs &B, const float *X, int n, float *yhat, hipStream_t s) {
    hipLaunchKernelGGL(mlp_tile_kernel<false>, dim3(mlp_groups(n, kMlpMaxForward)), dim3(kThreads), 0, s, B.params, B.mu, B.sd, X,
                       (const int *)nullptr, (const float *)nullptr, n, B.F, yhat, (float *)nullptr, (double *)nullptr);
    return hipGetLastError();
}

hipError_t mlp_train(const MlpBufs &B, const float *X, const float *y, const int *idx, int n, int t, float lr,
                     float *loss, hipStream_t s) {
    const unsigned groups = mlp_groups(n, kMlpGroups);
    hipLaunchKernelGGL(mlp_tile_kernel<true>, dim3(groups), dim3(kThreads), 0, s, B.params, B.mu, B.sd, X, idx, y, n, B.F,
                       (float *)nullptr, B.part, B.sqerr);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    const int P = mlp_nparams(B.F);
    Adam A{};
    if (t > 0) A = adam_args(B, t, lr);
    hipLaunchKernelGGL(mlp_reduce_kernel, dim3(param_blocks(P)), dim3(kThreads), 0, s, B.part, B.sqerr, (int)groups, P, n,
                       A, B.grad, loss);
    return hipGetLastError();
}

hipError_t mlp_adam(const MlpBufs &B, int t, float lr, hipStream_t s) {
    const int P = mlp_nparams(B.F);
    hipLaunchKernelGGL(mlp_adam_kernel, dim3(param_blocks(P)), dim3(kThreads), 0, s, adam_args(B, t, lr), B.grad, P);
    return hipGetLastError();
}

}  // namespace jk
