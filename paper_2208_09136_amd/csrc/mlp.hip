// mlp.hip -- the threshold-bracket network: a 66 -> 128 -> 128 -> 20
// perceptron with GELU hidden layers, its forward and backward passes, the
// mean-squared-error loss and Adam, as plain FP32 HIP kernels.
//
// The network maps the distance sketch of a series to the offsets
// t_r = (bits(eps_r) - scale) / 2^23 of its exact thresholds; it only
// narrows the key window in which exact selection looks (an extension of the
// method, not part of the paper).  Its arithmetic never decides a result:
// every threshold is still an exact order statistic.
//
// Parameter vector (float32, MLP_PARAMS entries):
//   W1 [IN][H], b1 [H], W2 [H][H], b2 [H], W3 [H][OUT], b3 [OUT]
// with W[i][o] at i * O + o.
//
// The layers are small (at most 128 x 128) and the calls latency-bound: what
// counts is the number of launches and the dependent round trips to L2 in
// each.  Every row's forward pass, loss and backward pass down to dZ1 depend
// on that row alone, so one kernel does them with the activations in LDS
// (k_rows), and a second forms all weight gradients (k_weights).  A training
// batch of 256 rows took nine launches and 266 us of kernels with a thread
// per output walking its whole dot product, and 294 us per call; now 53 us.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "mlp.h"

namespace rqa {

__device__ __forceinline__ float gelu(float z) { return 0.5f * z * (1.0f + erff(z * 0.70710678118654752f)); }

// d gelu / dz = Phi(z) + z phi(z)
__device__ __forceinline__ float gelu_grad(float z)
{
    return 0.5f * (1.0f + erff(z * 0.70710678118654752f)) + z * 0.39894228040143268f * expf(-0.5f * z * z);
}

// Rows of a k_rows workgroup, whose values of one unit form a float4 in LDS.
constexpr int ROWS = 4;
constexpr int ROWS_THREADS = 512;

__device__ __forceinline__ float4 fma4(float4 a, float w, float4 c)
{
    return make_float4(fmaf(a.x, w, c.x), fmaf(a.y, w, c.y), fmaf(a.z, w, c.z), fmaf(a.w, w, c.w));
}
__device__ __forceinline__ float4 add4(float4 a, float4 b)
{
    return make_float4(a.x + b.x, a.y + b.y, a.z + b.z, a.w + b.w);
}
__device__ __forceinline__ float at4(const float4& v, int r) { return r == 0 ? v.x : r == 1 ? v.y : r == 2 ? v.z : v.w; }

// Forward pass of ROWS rows; TRAIN: also the loss and the gradients dY, dZ2,
// dZ1 of the pre-activations.  Four groups of 128 threads share a hidden
// layer's dot products (a quarter of the inputs each, summed in group order),
// so that a layer waits for a quarter of the weight rows, loaded 11 to 32 at a
// time: 256 rows take 64 workgroups, 14 us forward and backward, where six
// launches of a thread per output took 66 us.
//   loss_partial[workgroup] = sum of (Y - T)^2 / (B OUT) over its rows.
template <bool TRAIN>
__global__ void __launch_bounds__(ROWS_THREADS)
k_rows(const float* __restrict__ P, const float* __restrict__ X, const float* __restrict__ T, int B,
       float* __restrict__ Y, MlpActs a, float* __restrict__ loss_partial)
{
    __shared__ float4 in[MLP_H], z1[MLP_H], z2[MLP_H], part[ROWS_THREADS];
    const MlpOffsets off;
    const int t = threadIdx.x, o = t & (MLP_H - 1), g = t / MLP_H;
    const int b0 = blockIdx.x * ROWS, nb = min(ROWS, B - b0);
    // the rows' inputs, transposed (rows past the batch are zero)
    if (t < MLP_IN) {
        float v[ROWS];
#pragma unroll
        for (int r = 0; r < ROWS; ++r) v[r] = r < nb ? X[(size_t)(b0 + r) * MLP_IN + t] : 0.f;
        in[t] = make_float4(v[0], v[1], v[2], v[3]);
    }
    __syncthreads();
    // one hidden layer: part -> z (pre-activations) -> in (activations)
    auto hidden = [&](int I, const float* W, const float* bias, float4* z, float* A) {
        const int per = (I + 3) / 4, i0 = g * per, i1 = min(i0 + per, I);
        float4 acc = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll 16
        for (int i = i0; i < i1; ++i) acc = fma4(in[i], W[(size_t)i * MLP_H + o], acc);
        part[t] = acc;
        __syncthreads();
        if (g == 0) {
            const float bo = bias[o];
            float4 s = add4(make_float4(bo, bo, bo, bo), part[o]);
#pragma unroll
            for (int h = 1; h < 4; ++h) s = add4(s, part[h * MLP_H + o]);
            z[o] = s;
            const float4 y = make_float4(gelu(s.x), gelu(s.y), gelu(s.z), gelu(s.w));
            in[o] = y;
            if constexpr (TRAIN) {
#pragma unroll
                for (int r = 0; r < ROWS; ++r)
                    if (r < nb) A[(size_t)(b0 + r) * MLP_H + o] = at4(y, r);
            }
        }
        __syncthreads();
    };
    hidden(MLP_IN, P + off.W1, P + off.b1, z1, a.A1);
    hidden(MLP_H, P + off.W2, P + off.b2, z2, a.A2);
    // output layer: sixteen groups of 32 threads, eight inputs each
    {
        const int q = t & 31, h = t >> 5;
        float4 acc = make_float4(0.f, 0.f, 0.f, 0.f);
        if (q < MLP_OUT) {
#pragma unroll
            for (int i = 0; i < 8; ++i) acc = fma4(in[8 * h + i], P[off.W3 + (size_t)(8 * h + i) * MLP_OUT + q], acc);
        }
        part[t] = acc;
        __syncthreads();
    }
    if (t < 64) {
        float e = 0.f;
        if (t < MLP_OUT) {
            const float bo = P[off.b3 + t];
            float4 s = make_float4(bo, bo, bo, bo);
#pragma unroll
            for (int h = 0; h < 16; ++h) s = add4(s, part[32 * h + t]);
            if constexpr (TRAIN) {
                const float n = (float)(B * MLP_OUT);
                float d[ROWS];
#pragma unroll
                for (int r = 0; r < ROWS; ++r) {
                    const size_t at = (size_t)(b0 + r) * MLP_OUT + t;
                    const float df = r < nb ? at4(s, r) - T[at] : 0.f;
                    d[r] = 2.0f * df / n;
                    e += df * df / n;
                    if (r < nb) a.dY[at] = d[r];
                }
                in[t] = make_float4(d[0], d[1], d[2], d[3]);
            } else {
#pragma unroll
                for (int r = 0; r < ROWS; ++r)
                    if (r < nb) Y[(size_t)(b0 + r) * MLP_OUT + t] = at4(s, r);
            }
        }
        if constexpr (TRAIN) {
#pragma unroll
            for (int m = 32; m > 0; m >>= 1) e += __shfl_xor(e, m);
            if (t == 0) loss_partial[blockIdx.x] = e;
        }
    }
    if constexpr (!TRAIN) return;
    __syncthreads();
    // dZ of the layer below: part = sum over a quarter of the outputs of in
    // (the gradients above, one float4 per output) times row i of W
    auto below = [&](int O, const float* W, const float4* z, float* dZ) {
        const int per = O / 4;
        const float4* w4 = (const float4*)(W + (size_t)o * O + g * per);
        float4 acc = make_float4(0.f, 0.f, 0.f, 0.f);
        if (per % 4 == 0) {
#pragma unroll 8
            for (int c = 0; c < per / 4; ++c) {
                const float4 w = w4[c];
                const float4* d = in + g * per + 4 * c;
                acc = fma4(d[3], w.w, fma4(d[2], w.z, fma4(d[1], w.y, fma4(d[0], w.x, acc))));
            }
        } else {
#pragma unroll 5
            for (int c = 0; c < per; ++c) acc = fma4(in[g * per + c], W[(size_t)o * O + g * per + c], acc);
        }
        part[t] = acc;
        __syncthreads();
        if (g == 0) {
            float4 s = part[o];
#pragma unroll
            for (int h = 1; h < 4; ++h) s = add4(s, part[h * MLP_H + o]);
            const float4 v = z[o];
            s = make_float4(s.x * gelu_grad(v.x), s.y * gelu_grad(v.y), s.z * gelu_grad(v.z), s.w * gelu_grad(v.w));
            in[o] = s;
#pragma unroll
            for (int r = 0; r < ROWS; ++r)
                if (r < nb) dZ[(size_t)(b0 + r) * MLP_H + o] = at4(s, r);
        }
        __syncthreads();
    };
    below(MLP_OUT, P + off.W3, z2, a.dZ2);
    below(MLP_H, P + off.W2, z1, a.dZ1);
}

// Weight gradients of all three layers: dW[i][o] = sum_b in[b][i] dZ[b][o] and
// the bias gradient sum_b dZ[b][o] as row I.  A workgroup of 16 waves forms a
// tile of WTILE rows x 64 columns; wave k sums the batch rows b = k mod 16 (its
// inputs are wave-uniform: one scalar load per row of the tile) and the waves'
// partial sums are added in wave order.  A thread per output walking all 256
// rows took 60 us per layer; the three layers here together 10 us.
constexpr int WTILE = 8;
constexpr int WAVES = 16;

struct LayerGrad {
    const float* in;   // [B][I]
    const float* dZ;   // [B][O]
    float* grad;       // dW [I][O], then db [O]
    int I, O, blocks;  // blocks = tiles of WTILE rows x 64 columns
};

__global__ void __launch_bounds__(64 * WAVES) k_weights(LayerGrad l0, LayerGrad l1, LayerGrad l2, int B)
{
    __shared__ float part[WAVES][WTILE][64];
    int blk = blockIdx.x;
    LayerGrad l = l0;
    if (blk >= l0.blocks) {
        blk -= l0.blocks;
        l = l1;
        if (blk >= l1.blocks) {
            blk -= l1.blocks;
            l = l2;
        }
    }
    const int cols = (l.O + 63) / 64;
    const int i0 = blk / cols * WTILE, o = blk % cols * 64 + (threadIdx.x & 63);
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const bool col = o < l.O;
    float acc[WTILE];
#pragma unroll
    for (int j = 0; j < WTILE; ++j) acc[j] = 0.f;
#pragma unroll 4
    for (int b = wave; b < B; b += WAVES) {
        const float dz = col ? l.dZ[(size_t)b * l.O + o] : 0.f;
        const float* x = l.in + (size_t)b * l.I;
#pragma unroll
        for (int j = 0; j < WTILE; ++j) {
            const int i = i0 + j;
            const float v = i < l.I ? x[i] : 1.f;
            acc[j] = fmaf(v, dz, acc[j]);
        }
    }
#pragma unroll
    for (int j = 0; j < WTILE; ++j) part[wave][j][threadIdx.x & 63] = acc[j];
    __syncthreads();
    const int j = threadIdx.x >> 6;
    if (j < WTILE && i0 + j <= l.I && col) {
        float s = 0.f;
#pragma unroll
        for (int k = 0; k < WAVES; ++k) s += part[k][j][threadIdx.x & 63];
        l.grad[(size_t)(i0 + j) * l.O + o] = s;
    }
}

// Adam (Kingma and Ba): m = b1 m + (1-b1) g, v = b2 v + (1-b2) g^2,
// theta -= lr * (m / c1) / (sqrt(v / c2) + eps) with c1 = 1 - b1^t, c2 = 1 - b2^t.
__global__ void k_adam(float* __restrict__ th, const float* __restrict__ g, float* __restrict__ m,
                       float* __restrict__ v, int n, float lr, float b1, float b2, float eps, float c1, float c2)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const float gi = g[i];
    const float mi = b1 * m[i] + (1.f - b1) * gi;
    const float vi = b2 * v[i] + (1.f - b2) * gi * gi;
    m[i] = mi;
    v[i] = vi;
    th[i] -= lr * (mi / c1) / (sqrtf(vi / c2) + eps);
}

static inline unsigned blocks(long n, int t) { return (unsigned)((n + t - 1) / t); }

hipError_t mlp_forward(hipStream_t st, const float* params, const float* X, int B, float* Y)
{
    hipLaunchKernelGGL(k_rows<false>, dim3(blocks(B, ROWS)), dim3(ROWS_THREADS), 0, st, params, X, (const float*)nullptr, B,
                       Y, MlpActs{}, (float*)nullptr);
    return hipGetLastError();
}

int mlp_loss_partials(int B) { return (int)blocks(B, ROWS); }

hipError_t mlp_gradients(hipStream_t st, const float* params, const float* X, const float* T, int B, const MlpActs& a,
                         float* grad, float* loss_partial)
{
    const MlpOffsets o;
    static_assert(sizeof(float) * 4 == sizeof(float4), "weight rows are read four floats at a time");
    hipLaunchKernelGGL(k_rows<true>, dim3(blocks(B, ROWS)), dim3(ROWS_THREADS), 0, st, params, X, T, B, (float*)nullptr, a,
                       loss_partial);
    auto layer = [](const float* in, const float* dZ, float* g, int I, int O) {
        return LayerGrad{in, dZ, g, I, O, (I + WTILE) / WTILE * ((O + 63) / 64)};
    };
    // the bias gradient follows the weights of its layer in the parameter vector
    const LayerGrad l0 = layer(a.A1, a.dZ2, grad + o.W2, MLP_H, MLP_H), l1 = layer(X, a.dZ1, grad + o.W1, MLP_IN, MLP_H),
                    l2 = layer(a.A2, a.dY, grad + o.W3, MLP_H, MLP_OUT);
    hipLaunchKernelGGL(k_weights, dim3(l0.blocks + l1.blocks + l2.blocks), dim3(64 * WAVES), 0, st, l0, l1, l2, B);
    return hipGetLastError();
}

hipError_t mlp_adam(hipStream_t st, float* params, const float* grad, float* m, float* v, float lr, float b1,
                    float b2, float eps, float c1, float c2)
{
    hipLaunchKernelGGL(k_adam, dim3(blocks(MLP_PARAMS, 256)), dim3(256), 0, st, params, grad, m, v, MLP_PARAMS, lr, b1,
                       b2, eps, c1, c2);
    return hipGetLastError();
}

}  // namespace rqa
