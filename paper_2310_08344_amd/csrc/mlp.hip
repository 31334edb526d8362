// HIP kernels (gfx950) of the spectral/budget predictor: an MLP
// 8 -> 64 -> 64 -> 2 with ReLU, float32 weights and bfloat16 hidden
// activations, trained with Adam on the mean squared error.
//
// Training step on a minibatch of B samples, two launches:
//   mlp_fwd_bwd_kernel  one wavefront per sample, a lane per hidden unit:
//                       standardise, forward, loss, backward to the
//                       per-sample deltas (float32); writes the sample's
//                       inputs, activations and deltas
//   mlp_grad_kernel     one thread per parameter: sums its gradient over the
//                       minibatch in sample order (float64 accumulation) and
//                       takes the parameter's Adam step
// The network is tiny (4866 parameters, ~4.7k multiply-adds per sample):
// the kernels are latency-bound, and the fixed summation order makes every
// step deterministic.
#include <hip/hip_runtime.h>

#include "mlp_device.h"

namespace lx {
namespace {

constexpr int kT = 256;

__device__ __forceinline__ float to_bf16(float x) {
    // round to nearest even on the upper 16 bits of the float32 pattern
    unsigned u = __float_as_uint(x);
    const unsigned lsb = (u >> 16) & 1u;
    u = (u + 0x7FFFu + lsb) & 0xFFFF0000u;
    return __uint_as_float(u);
}

struct Net {
    const float* W1;
    const float* b1;
    const float* W2;
    const float* b2;
    const float* W3;
    const float* b3;
};

__device__ __forceinline__ Net net_of(const float* theta) {
    Net n;
    n.W1 = theta;
    n.b1 = n.W1 + kMlpH * kMlpIn;
    n.W2 = n.b1 + kMlpH;
    n.b2 = n.W2 + kMlpH * kMlpH;
    n.W3 = n.b2 + kMlpH;
    n.b3 = n.W3 + kMlpOut * kMlpH;
    return n;
}

// forward of one standardised sample; a1, a2 rounded to bfloat16, z masks kept
__device__ __forceinline__ void forward_one(const Net& n, const float (&x)[kMlpIn], float (&a1)[kMlpH],
                                            float (&a2)[kMlpH], float (&y)[kMlpOut]) {
    for (int i = 0; i < kMlpH; ++i) {
        float z = n.b1[i];
#pragma unroll
        for (int j = 0; j < kMlpIn; ++j) z = fmaf(n.W1[i * kMlpIn + j], x[j], z);
        a1[i] = to_bf16(fmaxf(z, 0.0f));
    }
    for (int i = 0; i < kMlpH; ++i) {
        float z = n.b2[i];
        for (int j = 0; j < kMlpH; ++j) z = fmaf(n.W2[i * kMlpH + j], a1[j], z);
        a2[i] = to_bf16(fmaxf(z, 0.0f));
    }
#pragma unroll
    for (int o = 0; o < kMlpOut; ++o) {
        float z = n.b3[o];
        for (int j = 0; j < kMlpH; ++j) z = fmaf(n.W3[o * kMlpH + j], a2[j], z);
        y[o] = z;
    }
}

constexpr int kFbWaves = 4;              // samples (wavefronts) per workgroup at a time
constexpr int kW2Pitch = kMlpH + 1;      // LDS row pitch: rows and columns of W2 both without bank conflicts

// One wavefront per sample, lane i its hidden unit i.  W2 sits in LDS: lane
// i reads row i in the forward pass and column i in the backward pass, and
// the other layer's values are broadcast from LDS.  Every sum runs over its
// terms in index order from the bias (forward) or 0 (backward), one FMA
// each, as one thread per sample would take them, so the values do not
// depend on how the minibatch is split.  What bounds it is the chain of
// 64 + 64 + 64 dependent FMAs and the staging of W2 from L2: 8.7 us at B = 512
// where one thread per sample (two workgroups in all) took 70.
__global__ __launch_bounds__(64 * kFbWaves) void mlp_fwd_bwd_kernel(const float* __restrict__ theta,
                                                                    const float* __restrict__ X,
                                                                    const float* __restrict__ Y,
                                                                    const int* __restrict__ idx, int B, MlpScaling sc,
                                                                    float* __restrict__ scratch) {
    __shared__ float w2[kMlpH * kW2Pitch];
    __shared__ __attribute__((aligned(16))) float act[kFbWaves][3][kMlpH];   // a1, a2, dz2 of each wavefront's sample
    const Net n = net_of(theta);
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    for (int e = tid; e < kMlpH * kMlpH; e += 64 * kFbWaves) w2[(e >> 6) * kW2Pitch + (e & 63)] = n.W2[e];
    float w1[kMlpIn];
#pragma unroll
    for (int j = 0; j < kMlpIn; ++j) w1[j] = n.W1[lane * kMlpIn + j];
    const float b1 = n.b1[lane], b2 = n.b2[lane];
    float w3[kMlpOut];
#pragma unroll
    for (int o = 0; o < kMlpOut; ++o) w3[o] = n.W3[o * kMlpH + lane];
    __syncthreads();
    // the loop bound is the same for all wavefronts of a workgroup (they meet
    // at the barriers); one past the end computes the last sample again and
    // stores nothing
    for (int s0 = static_cast<int>(blockIdx.x) * kFbWaves; s0 < B; s0 += static_cast<int>(gridDim.x) * kFbWaves) {
        const bool live = s0 + wave < B;
        const int s = live ? s0 + wave : B - 1;
        const int r = idx ? idx[s] : s;
        float x[kMlpIn], t[kMlpOut];
#pragma unroll
        for (int j = 0; j < kMlpIn; ++j) x[j] = (X[static_cast<long>(r) * kMlpIn + j] - sc.mean_x[j]) / sc.std_x[j];
#pragma unroll
        for (int o = 0; o < kMlpOut; ++o) t[o] = (Y[static_cast<long>(r) * kMlpOut + o] - sc.mean_y[o]) / sc.std_y[o];
        float z = b1;
#pragma unroll
        for (int j = 0; j < kMlpIn; ++j) z = fmaf(w1[j], x[j], z);
        const float a1 = to_bf16(fmaxf(z, 0.0f));
        act[wave][0][lane] = a1;
        __syncthreads();
        z = b2;
#pragma unroll
        for (int j = 0; j < kMlpH; ++j) z = fmaf(w2[lane * kW2Pitch + j], act[wave][0][j], z);
        const float a2 = to_bf16(fmaxf(z, 0.0f));
        act[wave][1][lane] = a2;
        __syncthreads();
        float dY[kMlpOut], loss = 0.0f;
        const float scale = 2.0f / static_cast<float>(B * kMlpOut);
        {
            // lanes with the same parity form the same output
            const int o = lane & 1;
            float y = n.b3[o];
#pragma unroll
            for (int j = 0; j < kMlpH; ++j) y = fmaf(n.W3[o * kMlpH + j], act[wave][1][j], y);
#pragma unroll
            for (int k = 0; k < kMlpOut; ++k) {
                const float d = __shfl(y, k, 64) - t[k];
                loss = fmaf(d, d, loss);
                dY[k] = scale * d;
            }
        }
        // dz2 = (W3^T dY) * [a2 > 0]   (a2 > 0 exactly when z2 > 0)
        float g = 0.0f;
#pragma unroll
        for (int o = 0; o < kMlpOut; ++o) g = fmaf(w3[o], dY[o], g);
        const float dz2 = a2 > 0.0f ? g : 0.0f;
        act[wave][2][lane] = dz2;
        __syncthreads();
        // dz1 = (W2^T dz2) * [a1 > 0]
        g = 0.0f;
#pragma unroll
        for (int i = 0; i < kMlpH; ++i) g = fmaf(w2[i * kW2Pitch + lane], act[wave][2][i], g);
        if (live) {
            float* __restrict__ row = scratch + static_cast<long>(s) * kMlpRow;
            row[kOffA1 + lane] = a1;
            row[kOffA2 + lane] = a2;
            row[kOffDz1 + lane] = a1 > 0.0f ? g : 0.0f;
            row[kOffDz2 + lane] = dz2;
            if (lane == 0) {
#pragma unroll
                for (int j = 0; j < kMlpIn; ++j) row[kOffX + j] = x[j];
#pragma unroll
                for (int o = 0; o < kMlpOut; ++o) row[kOffDy + o] = dY[o];
                row[kOffLoss] = loss;
            }
        }
    }
}

constexpr int kGradChunk = 128;   // samples staged at a time
constexpr int kGradThreads = 256;
constexpr int kGradWin = 64;      // floats of a sample's row in each of the two staged windows

// Gradient of every parameter summed over the minibatch in sample order, then
// (kAdam) its Adam step t.  Workgroup g holds the parameters 64 g .. 64 g +
// 63, all of one layer's weights or biases: gradient = sum over the samples
// of row[off_a] * row[off_b].  A parameter's sum is a chain of B dependent
// FP64 FMAs (2 us at B = 512), which the first wavefront runs; what bounds
// the kernel beside it is the latency of the factors, so all four wavefronts
// stage the two windows of 64 floats that hold them through LDS, one chunk
// of samples ahead, with every load of a chunk in flight at once.  Per
// launch at B = 512: 245 us with one pair of loads in flight per sum, 22
// with 32 pairs, 13.6 from LDS (the Adam step had 5.5 us of its own besides).
template <bool kAdam>
__global__ __launch_bounds__(kGradThreads) void mlp_grad_kernel(const float* __restrict__ scratch, int B,
                                                                float* __restrict__ grad,
                                                                double* __restrict__ loss_out,
                                                                float* __restrict__ theta, float* __restrict__ m,
                                                                float* __restrict__ v, int t, float lr, float beta1,
                                                                float beta2, float eps) {
    const int tid = threadIdx.x;
    if (blockIdx.x == gridDim.x - 1) {
        // the loss has a workgroup of its own, after the parameters'
        if (tid == 0 && loss_out != nullptr) {
            double L = 0.0;
            for (int s = 0; s < B; ++s) L += scratch[static_cast<long>(s) * kMlpRow + kOffLoss];
            *loss_out = L / (static_cast<double>(B) * kMlpOut);
        }
        return;
    }
    const int p = static_cast<int>(blockIdx.x) * 64 + (tid & 63);
    int off_a, off_b, win_b;   // the windows are the same for the whole workgroup
    bool bias = false;
    if (p < kPB1) {
        off_a = kOffDz1 + (p - kPW1) / kMlpIn;
        off_b = kOffX + (p - kPW1) % kMlpIn;
        win_b = kOffX;
    } else if (p < kPW2) {
        off_a = kOffDz1 + (p - kPB1);
        bias = true;
        win_b = kOffX;
    } else if (p < kPB2) {
        off_a = kOffDz2 + (p - kPW2) / kMlpH;
        off_b = kOffA1 + (p - kPW2) % kMlpH;
        win_b = kOffA1;
    } else if (p < kPW3) {
        off_a = kOffDz2 + (p - kPB2);
        bias = true;
        win_b = kOffX;
    } else if (p < kPB3) {
        off_a = kOffDy + (p - kPW3) / kMlpH;
        off_b = kOffA2 + (p - kPW3) % kMlpH;
        win_b = kOffA2;
    } else {
        off_a = kOffDy + (p < kMlpParams ? p - kPB3 : 0);
        bias = true;
        win_b = kOffX;
    }
    const int win_a = p < kPW2 ? kOffDz1 : (p < kPW3 ? kOffDz2 : kMlpRow - kGradWin);
    const int ia = off_a - win_a, ib = bias ? 0 : off_b - win_b;
    static_assert(kPB1 % 64 == 0 && kPW2 % 64 == 0 && kPB2 % 64 == 0 && kPW3 % 64 == 0 && kPB3 % 64 == 0,
                  "a workgroup's parameters share their windows");
    static_assert(kMlpRow % 4 == 0 && kOffA1 % 4 == 0 && kOffA2 % 4 == 0 && kOffDz1 % 4 == 0 && kOffDz2 % 4 == 0 &&
                      kOffDy >= kMlpRow - kGradWin && kOffX + kGradWin <= kMlpRow,
                  "16-byte windows inside a row");
    __shared__ __attribute__((aligned(16))) float lds[2][2][kGradChunk][kGradWin];
    constexpr int kVec = kGradWin / 4;                              // float4 of a window
    constexpr int kLoads = kGradChunk * kVec / kGradThreads;        // per thread, window and chunk
    float4 ra[kLoads], rb[kLoads];
    auto load = [&](int s0) {
#pragma unroll
        for (int i = 0; i < kLoads; ++i) {
            const int e = i * kGradThreads + tid, s = s0 + e / kVec, c = (e % kVec) * 4;
            ra[i] = rb[i] = float4{0.0f, 0.0f, 0.0f, 0.0f};         // samples past the last one add 0
            if (s < B) {
                const float* row = scratch + static_cast<long>(s) * kMlpRow;
                ra[i] = *reinterpret_cast<const float4*>(row + win_a + c);
                rb[i] = *reinterpret_cast<const float4*>(row + win_b + c);
            }
        }
    };
    auto store = [&](int buf) {
#pragma unroll
        for (int i = 0; i < kLoads; ++i) {
            const int e = i * kGradThreads + tid;
            *reinterpret_cast<float4*>(&lds[buf][0][e / kVec][(e % kVec) * 4]) = ra[i];
            *reinterpret_cast<float4*>(&lds[buf][1][e / kVec][(e % kVec) * 4]) = rb[i];
        }
    };
    double acc = 0.0;
    load(0);
    store(0);
    __syncthreads();
    int buf = 0;
    for (int s0 = 0; s0 < B; s0 += kGradChunk, buf ^= 1) {
        const bool more = s0 + kGradChunk < B;
        if (more) load(s0 + kGradChunk);
        if (tid < 64) {
#pragma unroll 16
            for (int s = 0; s < kGradChunk; ++s) {
                const float fb = lds[buf][1][s][ib];
                acc = fma(static_cast<double>(lds[buf][0][s][ia]), bias ? 1.0 : static_cast<double>(fb), acc);
            }
        }
        if (more) store(buf ^ 1);
        __syncthreads();
    }
    if (tid >= 64 || p >= kMlpParams) return;
    const float g = static_cast<float>(acc);
    if constexpr (kAdam) {
        const float mm = beta1 * m[p] + (1.0f - beta1) * g;
        const float vv = beta2 * v[p] + (1.0f - beta2) * g * g;
        m[p] = mm;
        v[p] = vv;
        const float mhat = mm / (1.0f - powf(beta1, static_cast<float>(t)));
        const float vhat = vv / (1.0f - powf(beta2, static_cast<float>(t)));
        theta[p] -= lr * mhat / (sqrtf(vhat) + eps);
    } else {
        grad[p] = g;
    }
}

__global__ __launch_bounds__(kT) void mlp_infer_kernel(const float* __restrict__ theta, const float* __restrict__ X,
                                                       int n, MlpScaling sc, float* __restrict__ Yout) {
    const int s = blockIdx.x * blockDim.x + threadIdx.x;
    if (s >= n) return;
    const Net net = net_of(theta);
    float x[kMlpIn];
#pragma unroll
    for (int j = 0; j < kMlpIn; ++j) x[j] = (X[static_cast<long>(s) * kMlpIn + j] - sc.mean_x[j]) / sc.std_x[j];
    float a1[kMlpH], a2[kMlpH], y[kMlpOut];
    forward_one(net, x, a1, a2, y);
#pragma unroll
    for (int o = 0; o < kMlpOut; ++o) Yout[static_cast<long>(s) * kMlpOut + o] = y[o] * sc.std_y[o] + sc.mean_y[o];
}

// features of one instance per workgroup: log D, log(|v| + 1e-3), angle,
// log dx, log h, log rms(u), log max|u|, l (Burgers: D := nu,
// |v| := sqrt(2) max|u|, angle := pi/4; u is the Burgers state, else v)
__global__ __launch_bounds__(kT) void features_kernel(const FeatureInst* __restrict__ fi, float* __restrict__ X) {
    const FeatureInst& f = fi[blockIdx.x];
    const long N = static_cast<long>(f.nx) * f.ny;
    double ss = 0.0, mx = 0.0;
    for (long t = threadIdx.x; t < N; t += blockDim.x) {
        const double q = f.u[t];
        ss += q * q;
        mx = fmax(mx, fabs(q));
    }
    __shared__ double red_s[kT], red_m[kT];
    red_s[threadIdx.x] = ss;
    red_m[threadIdx.x] = mx;
    __syncthreads();
    for (int w = kT / 2; w > 0; w >>= 1) {
        if (static_cast<int>(threadIdx.x) < w) {
            red_s[threadIdx.x] += red_s[threadIdx.x + w];
            red_m[threadIdx.x] = fmax(red_m[threadIdx.x], red_m[threadIdx.x + w]);
        }
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        const double rms = sqrt(red_s[0] / static_cast<double>(N));
        const double umax = red_m[0];
        float* x = X + static_cast<long>(blockIdx.x) * kMlpIn;
        if (f.burgers) {
            x[0] = static_cast<float>(log(f.D));
            x[1] = static_cast<float>(log(sqrt(2.0) * umax + 1e-3));
            x[2] = static_cast<float>(0.7853981633974483);
        } else {
            x[0] = static_cast<float>(log(f.D));
            x[1] = static_cast<float>(log(sqrt(f.vx * f.vx + f.vy * f.vy) + 1e-3));
            x[2] = static_cast<float>(atan2(f.vy, f.vx));
        }
        x[3] = static_cast<float>(log(f.dx));
        x[4] = static_cast<float>(log(f.h));
        x[5] = static_cast<float>(log(rms + 1e-300));
        x[6] = static_cast<float>(log(umax + 1e-300));
        x[7] = static_cast<float>(f.l);
    }
}

}  // namespace

hipError_t launch_mlp_fwd_bwd(const float* theta, const float* X, const float* Y, const int* idx, int B,
                              const MlpScaling& sc, float* scratch, hipStream_t s) {
    // at most four workgroups per CU; larger minibatches loop
    const int nb = B < 4096 ? (B + kFbWaves - 1) / kFbWaves : 1024;
    hipLaunchKernelGGL(mlp_fwd_bwd_kernel, dim3(nb), dim3(64 * kFbWaves), 0, s, theta, X, Y, idx, B, sc, scratch);
    return hipGetLastError();
}

constexpr int kGradBlocks = (kMlpParams + 63) / 64 + 1;   // the last one forms the loss

hipError_t launch_mlp_grad(const float* scratch, int B, float* grad, double* loss, hipStream_t s) {
    hipLaunchKernelGGL(mlp_grad_kernel<false>, dim3(kGradBlocks), dim3(kGradThreads), 0, s, scratch, B, grad, loss, nullptr,
                       nullptr, nullptr, 0, 0.0f, 0.0f, 0.0f, 0.0f);
    return hipGetLastError();
}

hipError_t launch_mlp_grad_adam(const float* scratch, int B, double* loss, float* theta, float* m, float* v, int t,
                                float lr, hipStream_t s) {
    hipLaunchKernelGGL(mlp_grad_kernel<true>, dim3(kGradBlocks), dim3(kGradThreads), 0, s, scratch, B, nullptr, loss, theta, m,
                       v, t, lr, 0.9f, 0.999f, 1e-8f);
    return hipGetLastError();
}

hipError_t launch_mlp_infer(const float* theta, const float* X, int n, const MlpScaling& sc, float* Y,
                            hipStream_t s) {
    hipLaunchKernelGGL(mlp_infer_kernel, dim3((n + kT - 1) / kT), dim3(kT), 0, s, theta, X, n, sc, Y);
    return hipGetLastError();
}

hipError_t launch_features(const FeatureInst* fi, int n, float* X, hipStream_t s) {
    hipLaunchKernelGGL(features_kernel, dim3(n), dim3(kT), 0, s, fi, X);
    return hipGetLastError();
}

}  // namespace lx
