// Kernels of the learned threshold: tile-norm histogram features, norm
// product bounds, FP64 sums of squares (for relative errors), and the
// training and inference kernels of the 129-128-128-1 GELU network.
//
// All reductions run in a fixed order, so every result is bitwise
// reproducible from run to run.
#include <hip/hip_runtime.h>

#include <cmath>

#include "internal.h"

namespace spamm {

// --------------------------------------------------------------------------
// Features: per matrix a 64-bin histogram of log10 of the positive leaf norms
// over [-46, 3) (norms outside the range in the first or last bin), as tiles
// per tile row (count / bdim) capped at kHistCap; zero norms are not
// counted.  Then log10(target).

constexpr int kHistBins = 64;
constexpr double kLogLo = -46.0, kLogHi = 3.0;
constexpr double kHistCap = 4.0;
constexpr int kFeatThreads = 1024;

__global__ __launch_bounds__(kFeatThreads) void tau_features_kernel(const double* __restrict__ pyr_a,
                                                                    const double* __restrict__ pyr_b, int64_t bdim,
                                                                    int lv, float log_target,
                                                                    float* __restrict__ out) {
    __shared__ int hist[2][kHistBins];
    if (threadIdx.x < 2 * kHistBins) hist[threadIdx.x / kHistBins][threadIdx.x % kHistBins] = 0;
    __syncthreads();
    const int64_t side = int64_t(1) << lv;
    const int64_t tiles = bdim * bdim;
    for (int m = 0; m < 2; ++m) {
        const double* leaf = (m == 0 ? pyr_a : pyr_b) + level_offset(lv);
        for (int64_t t = threadIdx.x; t < tiles; t += kFeatThreads) {
            const double x = leaf[(t / bdim) * side + t % bdim];
            if (x > 0.0) {
                const double pos = (log10(x) - kLogLo) * (double(kHistBins) / (kLogHi - kLogLo));
                const double f = floor(pos);
                const int bin = f < 0.0 ? 0 : (f > kHistBins - 1 ? kHistBins - 1 : int(f));
                atomicAdd(&hist[m][bin], 1);
            }
        }
    }
    __syncthreads();
    if (threadIdx.x < 2 * kHistBins) {
        const double per_row = double(hist[threadIdx.x / kHistBins][threadIdx.x % kHistBins]) / double(bdim);
        out[threadIdx.x] = float(per_row < kHistCap ? per_row : kHistCap);
    }
    if (threadIdx.x == 0) out[2 * kHistBins] = log_target;
}

hipError_t launch_tau_features(const double* pyr_a, const double* pyr_b, int64_t bdim, int lv, float log_target,
                               float* out, hipStream_t s) {
    tau_features_kernel<<<1, kFeatThreads, 0, s>>>(pyr_a, pyr_b, bdim, lv, log_target, out);
    return hipGetLastError();
}

// --------------------------------------------------------------------------
// Sum of squares of an FP32 array in FP64 (squares are exact in FP64): a fixed
// grid of kSumBlocks blocks writes one partial each, then one block adds them
// in a fixed tree order.

constexpr int kSumThreads = 256;

template <int T>
__device__ double block_sum(double v, double* red) {
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) v += __shfl_xor(v, o);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
    __syncthreads();
    double tot = 0.0;
    if (threadIdx.x == 0)
        for (int w = 0; w < T / 64; ++w) tot += red[w];
    return tot;
}

__global__ __launch_bounds__(kSumThreads) void sumsq_partial_kernel(const float* __restrict__ x, int64_t count,
                                                                    double* __restrict__ partials) {
    __shared__ double red[kSumThreads / 64];
    const int64_t stride = int64_t(gridDim.x) * kSumThreads;
    double acc = 0.0;
    const bool vec = (reinterpret_cast<uintptr_t>(x) & 15u) == 0;
    if (vec) {
        const int64_t n4 = count / 4;
        const float4* x4 = reinterpret_cast<const float4*>(x);
        for (int64_t q = int64_t(blockIdx.x) * kSumThreads + threadIdx.x; q < n4; q += stride) {
            const float4 v = x4[q];
            acc += double(v.x) * v.x + double(v.y) * v.y + double(v.z) * v.z + double(v.w) * v.w;
        }
        for (int64_t q = n4 * 4 + int64_t(blockIdx.x) * kSumThreads + threadIdx.x; q < count; q += stride)
            acc += double(x[q]) * x[q];
    } else {
        for (int64_t q = int64_t(blockIdx.x) * kSumThreads + threadIdx.x; q < count; q += stride)
            acc += double(x[q]) * x[q];
    }
    const double tot = block_sum<kSumThreads>(acc, red);
    if (threadIdx.x == 0) partials[blockIdx.x] = tot;
}

__global__ __launch_bounds__(kSumThreads) void sum_partials_kernel(const double* __restrict__ partials, int np,
                                                                   double* __restrict__ out) {
    __shared__ double red[kSumThreads / 64];
    double acc = 0.0;
    for (int q = threadIdx.x; q < np; q += kSumThreads) acc += partials[q];
    const double tot = block_sum<kSumThreads>(acc, red);
    if (threadIdx.x == 0) *out = tot;
}

hipError_t launch_sumsq(const float* x, int64_t count, double* partials, double* out, hipStream_t s) {
    sumsq_partial_kernel<<<kSumBlocks, kSumThreads, 0, s>>>(x, count, partials);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    sum_partials_kernel<<<1, kSumThreads, 0, s>>>(partials, kSumBlocks, out);
    return hipGetLastError();
}

// --------------------------------------------------------------------------
// The network, FP32.  Parameters flat: W1 [128][129], b1 [128], W2 [128][128],
// b2 [128], w3 [128], b3 [1].  Layer l maps X [B][I] to Z = X W^T + b and
// H = gelu(Z) (erf form) for the hidden layers; the output layer has no
// activation.
//
// A minibatch (256 rows) is 0.04 GFLOP, so the step is bound by launches and
// by the latency inside each of them.  Two launches make the gradient: one
// runs a row through the whole network and back to dZ1 with both weight
// matrices in LDS (mlp_rows_kernel), the other forms every parameter gradient
// as a product over the batch on FP32 MFMA (mlp_weight_grad_kernel).  Batch
// 256, gradient and Adam step: 260 -> 19 us; with one launch per layer and
// direction 221 us of it were weight gradients that walked the batch one row
// at a time.

__device__ __forceinline__ float gelu_f(float z) { return 0.5f * z * (1.0f + erff(z * 0.70710678118654752f)); }

__device__ __forceinline__ float gelu_grad_f(float z) {
    return 0.5f * (1.0f + erff(z * 0.70710678118654752f)) + z * expf(-0.5f * z * z) * 0.39894228040143268f;
}

constexpr int kRowThreads = 512;
constexpr int kRowParts = kRowThreads / kMlpHid;          // input ranges summed by different threads
constexpr int kRowW = kMlpIn;                             // LDS row stride of both matrices (odd: no bank conflicts)
constexpr int kRowPart1 = (kMlpIn + kRowParts - 1) / kRowParts, kRowPart2 = kMlpHid / kRowParts;
constexpr int kRowLoads = (kMlpHid * kMlpIn + kRowThreads - 1) / kRowThreads;
constexpr int kRowBlocks = 256;  // one block per CU: both matrices fill its LDS

// Block b takes rows b*RB .. of the batch, then every gridDim.x*RB further.
// Thread (o, part) sums one range of the inputs of unit o for RB rows; the
// ranges are added in ascending order.  RB rows share each weight read, but
// the operand broadcasts grow with them, so RB is the smallest of 1, 2 and 4
// that gives every row a block of its own.  GRAD: also the residual and
// dZ2, dZ1, and what mlp_weight_grad_kernel reads (h1, h2, d1, d2, y, dy).
template <int RB, bool GRAD>
__global__ __launch_bounds__(kRowThreads) void mlp_rows_kernel(const float* __restrict__ params,
                                                               const float* __restrict__ x,
                                                               const float* __restrict__ t, int batch, MlpLayout P,
                                                               MlpLayout A, float* __restrict__ acts,
                                                               float* __restrict__ y) {
    typedef float rows_t __attribute__((ext_vector_type(RB)));
    __shared__ float w1s[kMlpHid * kRowW], w2s[kMlpHid * kRowW];
    __shared__ __attribute__((aligned(16))) float in[kMlpIn * RB];  // the layer's input, [unit][row]
    __shared__ __attribute__((aligned(16))) float part[kRowParts * kMlpHid * RB];
    __shared__ float outp[kMlpHid / 64][RB], dys[RB];
    const int tid = threadIdx.x, o = tid & (kMlpHid - 1), q = tid / kMlpHid;

    float w2r[kMlpHid * kMlpHid / kRowThreads];
    {
        float w1r[kRowLoads];
#pragma unroll
        for (int u = 0; u < kRowLoads; ++u) {
            const int e = tid + u * kRowThreads;
            w1r[u] = e < kMlpHid * kMlpIn ? params[P.w1 + e] : 0.0f;
        }
#pragma unroll
        for (int u = 0; u < kMlpHid * kMlpHid / kRowThreads; ++u) w2r[u] = params[P.w2 + tid + u * kRowThreads];
#pragma unroll
        for (int u = 0; u < kRowLoads; ++u) {
            const int e = tid + u * kRowThreads;
            if (e < kMlpHid * kMlpIn) w1s[e] = w1r[u];  // rows of kMlpIn = kRowW floats already
        }
    }
    const float bias1 = params[P.b1 + o], bias2 = params[P.b2 + o], w3 = params[P.w3 + o], b3 = params[P.b3];
    bool w2_staged = false;

    auto zero = [](rows_t& v) {
#pragma unroll
        for (int r = 0; r < RB; ++r) reinterpret_cast<float*>(&v)[r] = 0.0f;
    };
    for (int64_t r0 = int64_t(blockIdx.x) * RB; r0 < batch; r0 += int64_t(gridDim.x) * RB) {
        const int rows = batch - r0 < RB ? int(batch - r0) : RB;
        for (int e = tid; e < kMlpIn * RB; e += kRowThreads) {
            const int r = e / kMlpIn, i = e - r * kMlpIn;
            in[i * RB + r] = r < rows ? x[(r0 + r) * kMlpIn + i] : 0.0f;
        }
        __syncthreads();
        rows_t acc;
        // sum over one range of input units u0 .. u1 of w(u) * in[u]
        auto run = [&](int u0, int u1, auto weight) {
            zero(acc);
#pragma unroll 4
            for (int u = u0; u < u1; ++u) {
                const float w = weight(u);
                const rows_t v = *reinterpret_cast<const rows_t*>(in + u * RB);
#pragma unroll
                for (int r = 0; r < RB; ++r)
                    reinterpret_cast<float*>(&acc)[r] =
                        fmaf(w, reinterpret_cast<const float*>(&v)[r], reinterpret_cast<float*>(&acc)[r]);
            }
            *reinterpret_cast<rows_t*>(part + (q * kMlpHid + o) * RB) = acc;
            __syncthreads();
        };
        // thread (o, q) finishes rows q, q + kRowParts, ... of unit o
        auto total = [&](int r) {
            float s = part[o * RB + r];
#pragma unroll
            for (int p = 1; p < kRowParts; ++p) s += part[(p * kMlpHid + o) * RB + r];
            return s;
        };
        static_assert(RB <= kRowParts, "one row per thread and unit");
        const bool mine = q < RB;
        const bool live = q < rows;
        const int64_t at = (r0 + q) * kMlpHid + o;
        float z1 = 0.0f, z2 = 0.0f;

        run(q * kRowPart1, q * kRowPart1 + kRowPart1 < kMlpIn ? q * kRowPart1 + kRowPart1 : kMlpIn,
            [&](int u) { return w1s[o * kRowW + u]; });
        if (mine) {
            z1 = total(q) + bias1;
            const float h = gelu_f(z1);
            in[o * RB + q] = h;
            if (GRAD && live) acts[A.h1 + at] = h;
        }
        if (!w2_staged) {
#pragma unroll
            for (int u = 0; u < kMlpHid * kMlpHid / kRowThreads; ++u) {
                const int e = tid + u * kRowThreads;
                w2s[(e / kMlpHid) * kRowW + e % kMlpHid] = w2r[u];
            }
            w2_staged = true;
        }
        __syncthreads();
        run(q * kRowPart2, (q + 1) * kRowPart2, [&](int u) { return w2s[o * kRowW + u]; });
        if (mine) {
            z2 = total(q) + bias2;
            const float h = gelu_f(z2);
            if (GRAD && live) acts[A.h2 + at] = h;
            float s = h * w3;
#pragma unroll
            for (int off = 32; off >= 1; off >>= 1) s += __shfl_xor(s, off);
            if ((tid & 63) == 0) outp[o >> 6][q] = s;
        }
        __syncthreads();
        if (tid < rows) {
            float s = outp[0][tid];
#pragma unroll
            for (int w = 1; w < kMlpHid / 64; ++w) s += outp[w][tid];
            s += b3;
            if (!GRAD) {
                y[r0 + tid] = s;
            } else {
                const float dy = 2.0f * (s - t[r0 + tid]) / float(batch);
                acts[A.y + r0 + tid] = s;
                acts[A.dy + r0 + tid] = dy;
                dys[tid] = dy;
            }
        }
        if (GRAD) {
            __syncthreads();
            if (mine) {
                const float d = live ? dys[q] * w3 * gelu_grad_f(z2) : 0.0f;
                in[o * RB + q] = d;
                if (live) acts[A.d2 + at] = d;
            }
            __syncthreads();
            run(q * kRowPart2, (q + 1) * kRowPart2, [&](int u) { return w2s[u * kRowW + o]; });
            if (mine && live) acts[A.d1 + at] = total(q) * gelu_grad_f(z1);
        }
        __syncthreads();  // in, part and outp are reused
    }
}

// Parameter gradients from the rows kernel's arrays: per layer
// dW[o][i] = sum_b dZ[b][o] X[b][i] with X extended by a column of ones whose
// products are db.  One 16 x 16 tile of dW per block of four waves: wave w
// takes rows 16 s + 4 w .. + 3 of the batch in step s (v_mfma_f32_16x16x4f32,
// operands straight from L2, eight steps of loads in flight), and the four
// partial tiles are added in wave order.  The last block reduces the loss.
constexpr int kGradTiles = (kMlpIn + 1 + 15) / 16;           // column tiles of a layer with its ones column
constexpr int kGradRowTiles = kMlpHid / 16;
constexpr int kGradLayerBlocks = kGradRowTiles * kGradTiles;  // layers 1 and 2
constexpr int kGradBlocks = 2 * kGradLayerBlocks + kGradTiles + 1;

__global__ __launch_bounds__(256) void mlp_weight_grad_kernel(const float* __restrict__ x, const float* __restrict__ t,
                                                              int batch, MlpLayout P, MlpLayout A,
                                                              const float* __restrict__ acts,
                                                              float* __restrict__ grad, float* __restrict__ loss) {
    typedef float f4g __attribute__((ext_vector_type(4)));
    __shared__ float part[3][256];
    __shared__ double red[4];
    const int blk = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    if (blk == kGradBlocks - 1) {  // loss = mean (y - t)^2
        double acc = 0.0;
        for (int b = tid; b < batch; b += 256) {
            const float r = acts[A.y + b] - t[b];
            acc += double(r) * r;
        }
        const double tot = block_sum<256>(acc, red);
        if (tid == 0 && loss) *loss = float(tot / batch);
        return;
    }
    const int layer = blk < kGradLayerBlocks ? 1 : (blk < 2 * kGradLayerBlocks ? 2 : 3);
    const int e = layer == 3 ? blk - 2 * kGradLayerBlocks : blk % kGradLayerBlocks;
    const int o0 = (e / kGradTiles) * 16, i0 = (e % kGradTiles) * 16;
    const int in = layer == 1 ? kMlpIn : kMlpHid, outs = layer == 3 ? 1 : kMlpHid;
    const float* dz = acts + (layer == 1 ? A.d1 : layer == 2 ? A.d2 : A.dy);
    const float* xs = layer == 1 ? x : acts + (layer == 2 ? A.h1 : A.h2);
    const int c = lane & 15, g = lane >> 4;
    const int o = o0 + c, i = i0 + c;
    const bool o_in = o < outs, i_in = i < in, i_one = i == in;
    f4g acc = {0.0f, 0.0f, 0.0f, 0.0f};
    constexpr int U = 8;
    for (int b0 = 4 * wave + g; b0 - g < batch; b0 += 16 * U) {
        float av[U], bv[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int b = b0 + 16 * u;
            const bool in_b = b < batch;
            av[u] = (in_b && o_in) ? dz[int64_t(b) * outs + o] : 0.0f;
            bv[u] = (in_b && i_in) ? xs[int64_t(b) * in + i] : (in_b && i_one ? 1.0f : 0.0f);
        }
#pragma unroll
        for (int u = 0; u < U; ++u) acc = __builtin_amdgcn_mfma_f32_16x16x4f32(av[u], bv[u], acc, 0, 0, 0);
    }
    if (wave > 0) {
#pragma unroll
        for (int v = 0; v < 4; ++v) part[wave - 1][v * 64 + lane] = acc[v];
    }
    __syncthreads();
    if (wave != 0) return;
    float* dw = grad + (layer == 1 ? P.w1 : layer == 2 ? P.w2 : P.w3);
    float* db = grad + (layer == 1 ? P.b1 : layer == 2 ? P.b2 : P.b3);
#pragma unroll
    for (int v = 0; v < 4; ++v) {  // accumulator v of lane (c, g): row 4 g + v, column c
        const float s = ((acc[v] + part[0][v * 64 + lane]) + part[1][v * 64 + lane]) + part[2][v * 64 + lane];
        const int row = o0 + 4 * g + v;
        if (row >= outs) continue;
        if (i_in)
            dw[int64_t(row) * in + i] = s;
        else if (i_one)
            db[row] = s;
    }
}

// Adam with bias correction: m = b1 m + (1-b1) g; v = b2 v + (1-b2) g^2;
// p -= lr (m / c1) / (sqrt(v / c2) + eps), c1 = 1 - b1^t, c2 = 1 - b2^t.
__global__ void adam_kernel(float* __restrict__ p, const float* __restrict__ g, float* __restrict__ m,
                            float* __restrict__ v, int64_t count, float lr, float b1, float b2, float eps, float c1,
                            float c2) {
    const int64_t q = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
    if (q >= count) return;
    const float gq = g[q];
    const float mq = b1 * m[q] + (1.0f - b1) * gq;
    const float vq = b2 * v[q] + (1.0f - b2) * gq * gq;
    m[q] = mq;
    v[q] = vq;
    p[q] -= lr * (mq / c1) / (sqrtf(vq / c2) + eps);
}

namespace {
unsigned blocks_for(int64_t count, int threads) { return unsigned((count + threads - 1) / threads); }
}  // namespace

template <bool GRAD>
static hipError_t launch_mlp_rows(const float* params, const float* x, const float* t, int batch, float* acts,
                                  float* y, hipStream_t s) {
    const MlpLayout P{}, A = MlpLayout::acts(batch);
    const int rb = batch <= kRowBlocks ? 1 : (batch <= 2 * kRowBlocks ? 2 : 4);
    const unsigned need = blocks_for(batch, rb), blocks = need < unsigned(kRowBlocks) ? need : unsigned(kRowBlocks);
    if (rb == 1)
        mlp_rows_kernel<1, GRAD><<<blocks, kRowThreads, 0, s>>>(params, x, t, batch, P, A, acts, y);
    else if (rb == 2)
        mlp_rows_kernel<2, GRAD><<<blocks, kRowThreads, 0, s>>>(params, x, t, batch, P, A, acts, y);
    else
        mlp_rows_kernel<4, GRAD><<<blocks, kRowThreads, 0, s>>>(params, x, t, batch, P, A, acts, y);
    return hipGetLastError();
}

hipError_t launch_mlp_forward(const float* params, const float* x, int batch, float* acts, float* y, hipStream_t s) {
    return launch_mlp_rows<false>(params, x, nullptr, batch, acts, y, s);
}

hipError_t launch_mlp_loss_grad(const float* params, const float* x, const float* t, int batch, float* acts,
                                float* grad, float* loss, hipStream_t s) {
    const hipError_t e = launch_mlp_rows<true>(params, x, t, batch, acts, nullptr, s);
    if (e != hipSuccess) return e;
    mlp_weight_grad_kernel<<<kGradBlocks, 256, 0, s>>>(x, t, batch, MlpLayout{}, MlpLayout::acts(batch), acts, grad,
                                                       loss);
    return hipGetLastError();
}

hipError_t launch_adam(float* params, const float* grad, float* m, float* v, int64_t count, float lr, float b1,
                       float b2, float eps, float c1, float c2, hipStream_t s) {
    adam_kernel<<<blocks_for(count, 256), 256, 0, s>>>(params, grad, m, v, count, lr, b1, b2, eps, c1, c2);
    return hipGetLastError();
}

}  // namespace spamm
