// mlp.hip -- the work-item cost model: a 4 -> 64 -> 64 -> 64 -> 1 FP32
// multilayer perceptron with ReLU activations, trained on the GPU by the
// kernels below (forward, backward, Adam) on per-item kernel timings, and
// used to predict item costs for scheduling.  It never affects the counts.
//
// Parameter layout (one packed float array):
//   W1[64][4] b1[64] W2[64][64] b2[64] W3[64][64] b3[64] W4[64] b4
// Inputs are standardised with per-feature mean/std and the target (log2 of
// the item time) with its own mean/std; both are part of the model.
#include <math.h>
#include <stdio.h>
#include <string.h>

#include <random>
#include <vector>

#include "internal.h"

namespace fcfc {

constexpr int NF = 4, NH = 64;
constexpr int OFF_W1 = 0, OFF_B1 = OFF_W1 + NH * NF, OFF_W2 = OFF_B1 + NH, OFF_B2 = OFF_W2 + NH * NH,
              OFF_W3 = OFF_B2 + NH, OFF_B3 = OFF_W3 + NH * NH, OFF_W4 = OFF_B3 + NH, OFF_B4 = OFF_W4 + NH,
              NPARAM = OFF_B4 + 1;
constexpr int MB = 64;  // smallest minibatch that model_train takes

struct Model {
    float* params = nullptr;  // device NPARAM
    float* grad = nullptr;    // device NPARAM (+1 loss accumulator)
    float* m1 = nullptr;      // Adam moments
    float* m2 = nullptr;
    float* part = nullptr;    // partial gradients of GRAD_BLOCKS workgroups (allocated by the first gradient)
    float norm[10] = {0, 0, 0, 0, 1, 1, 1, 1, 0, 1};  // x mean[4], x std[4], y mean, y std
    int step = 0;
};

struct NormArgs {
    float xm[NF], xs[NF], ym, ys;
};

// Both kernels below give a wave 16 samples and keep the activations of the
// three layers in the result layout of v_mfma_f32_16x16x4_f32: lane l holds,
// for sample l % 16, the units 16 m + 4 (l / 16) + r in register r of block m.
// That is also the layout of the next product's B operand when its step (m, r)
// takes the four units 16 m + 4 g + r, g = 0..3, so no value moves between
// lanes from layer to layer; the weights lie in LDS in the order of the A
// operand, 16 bytes a lane for the four steps of a block.  All products
// accumulate in FP32.
typedef float f4 __attribute__((ext_vector_type(4)));
constexpr int MT = 16;             // samples per wave and pass
constexpr int FRAG = NH * NH;      // floats of one weight matrix in LDS
constexpr int FWD_WAVES = 4, GRAD_WAVES = 4;
constexpr int FWD_BLOCKS = 1024, GRAD_BLOCKS = 256;
constexpr int TSTRIDE = NH + 4;    // row stride of the transposition buffer (bank-conflict free both ways)

// weight (row o, column k) of a product's A operand in LDS
__device__ inline int frag_at(int o, int k) {
    return ((((o >> 4) * 4 + (k >> 4)) * 64 + ((k >> 2) & 3) * 16 + (o & 15)) << 2) + (k & 3);
}

// out = init + A in, 64 x 64 by 64 x 16
__device__ __attribute__((always_inline)) inline void mlp_product(const float* F, int lane, const f4 in[4],
                                                                  f4 out[4]) {
#pragma unroll
    for (int m = 0; m < 4; m++) {
        f4 a[4];
#pragma unroll
        for (int o = 0; o < 4; o++) a[o] = ((const f4*)F)[(o * 4 + m) * 64 + lane];
#pragma unroll
        for (int r = 0; r < 4; r++)
#pragma unroll
            for (int o = 0; o < 4; o++) out[o] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[o][r], in[m][r], out[o], 0, 0, 0);
        __builtin_amdgcn_sched_barrier(0);  // at most 16 weights in flight: four waves fit where two would
    }
}

__device__ inline void relu(f4 h[4]) {
#pragma unroll
    for (int m = 0; m < 4; m++)
#pragma unroll
        for (int r = 0; r < 4; r++) h[m][r] = fmaxf(h[m][r], 0.f);
}

// the three hidden layers and the output of the wave's samples; x: feature
// lane / 16 of sample lane % 16, w1: W1[16 o + lane % 16][lane / 16]; V: b1, b2,
// b3, W4 in LDS
__device__ __attribute__((always_inline)) inline float mlp_layers(const float* F2, const float* F3, const float* V,
                                                                  const float w1[4], float b4, float x, int lane,
                                                                  f4 h1[4], f4 h2[4], f4 h3[4]) {
    const f4* v = (const f4*)V + (lane >> 4);
#pragma unroll
    for (int m = 0; m < 4; m++) {
        h1[m] = __builtin_amdgcn_mfma_f32_16x16x4f32(w1[m], x, v[m * 4], 0, 0, 0);
        h2[m] = v[16 + m * 4];
        h3[m] = v[32 + m * 4];
    }
    relu(h1);
    mlp_product(F2, lane, h1, h2);
    relu(h2);
    mlp_product(F3, lane, h2, h3);
    relu(h3);
    float y = 0.f;
#pragma unroll
    for (int m = 0; m < 4; m++) {
        const f4 w4 = v[48 + m * 4];
#pragma unroll
        for (int r = 0; r < 4; r++) y = __builtin_fmaf(w4[r], h3[m][r], y);
    }
    y += __shfl_xor(y, 16);
    y += __shfl_xor(y, 32);
    return y + b4;
}

// y[i] = ys * mlp((x[i] - xm) / xs) + ym.  Bound by the FP32 matrix rate (8.4k
// multiply-adds a sample).  MI355X, 500,009 samples: 0.16 -> 0.083 ms, 102
// TFLOP/s.
__global__ __launch_bounds__(64 * FWD_WAVES) void k_mlp_forward(const float* __restrict__ params,
                                                                const float* __restrict__ X, int64_t m, NormArgs nrm,
                                                                float* __restrict__ Y) {
    __shared__ __align__(16) float F2[FRAG], F3[FRAG], V[4 * NH];
    const int t = threadIdx.x, lane = t & 63, g = lane >> 4, c = lane & 15;
    for (int e = t; e < FRAG; e += 64 * FWD_WAVES) {
        const int at = frag_at(e / NH, e % NH);
        F2[at] = params[OFF_W2 + e];
        F3[at] = params[OFF_W3 + e];
    }
    for (int e = t; e < NH; e += 64 * FWD_WAVES) {
        V[e] = params[OFF_B1 + e];
        V[NH + e] = params[OFF_B2 + e];
        V[2 * NH + e] = params[OFF_B3 + e];
        V[3 * NH + e] = params[OFF_W4 + e];
    }
    float w1[4];
#pragma unroll
    for (int o = 0; o < 4; o++) w1[o] = params[OFF_W1 + (16 * o + c) * NF + g];
    const float b4 = params[OFF_B4];
    const float xm = g == 0 ? nrm.xm[0] : g == 1 ? nrm.xm[1] : g == 2 ? nrm.xm[2] : nrm.xm[3];
    const float xs = g == 0 ? nrm.xs[0] : g == 1 ? nrm.xs[1] : g == 2 ? nrm.xs[2] : nrm.xs[3];
    __syncthreads();
    const int64_t tiles = (m + MT - 1) / MT, step = (int64_t)gridDim.x * FWD_WAVES;
    int64_t tile = (int64_t)blockIdx.x * FWD_WAVES + (t >> 6);
    float xn = 0.f;
    if (tile < tiles && tile * MT + c < m) xn = X[(tile * MT + c) * NF + g];
    for (; tile < tiles; tile += step) {
        const int64_t s = tile * MT + c;
        const float x = (xn - xm) / xs;
        const int64_t sn = s + step * MT;
        if (sn < m) xn = X[sn * NF + g];
        f4 h1[4], h2[4], h3[4];
        const float y = mlp_layers(F2, F3, V, w1, b4, x, lane, h1, h2, h3);
        if (g == 0 && s < m) Y[s] = y * nrm.ys + nrm.ym;
    }
}

// orders the wave's LDS accesses
__device__ inline void wave_fence() {
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

// The wave's 64 x 16 activations with the samples along the steps of a product:
// out[m][r] = unit 16 m + lane % 16 of sample 4 (lane / 16) + r.
__device__ __attribute__((always_inline)) inline void mlp_transpose(float* T, int lane, const f4 in[4], f4 out[4]) {
    const int g = lane >> 4, c = lane & 15;
#pragma unroll
    for (int m = 0; m < 4; m++) *(f4*)(T + c * TSTRIDE + 16 * m + 4 * g) = in[m];
    wave_fence();
#pragma unroll
    for (int m = 0; m < 4; m++)
#pragma unroll
        for (int r = 0; r < 4; r++) out[m][r] = T[(4 * g + r) * TSTRIDE + 16 * m + c];
    wave_fence();
}

// g += a b^T over the wave's samples (a, b as mlp_transpose gives them)
__device__ __attribute__((always_inline)) inline void mlp_outer(const f4 a[4], const f4 b[4], f4 g[4][4]) {
#pragma unroll
    for (int r = 0; r < 4; r++)
#pragma unroll
        for (int o = 0; o < 4; o++)
#pragma unroll
            for (int i = 0; i < 4; i++)
                g[o][i] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[o][r], b[i][r], g[o][i], 0, 0, 0);
}

// Gradient of 0.5 * sum_s (y_s - t_s)^2 (standardised units) over samples
// [s0, s0 + count) taken through the permutation `perm` (or identity): each
// workgroup writes its partial sums (entry NPARAM: the loss) to row blockIdx.x
// of part[], which k_grad_sum adds up.  A wave keeps the gradient of both 64 x
// 64 layers in 128 accumulator registers over all its samples and takes the
// whole register file of its SIMD (two waves of 256 registers spilled 215);
// the samples reach the steps of those products through a transposition in
// LDS (a second set of products in the other orientation would add 67 % matrix
// work).  Bound by the FP32 matrix rate (25k multiply-adds a sample) and, with
// one wave, by the vector work between the products (two groups of samples a
// pass, sharing the weights read from LDS, ran the same).  MI355X, 500,009 samples:
// 7.2 -> 0.29 ms, 88 TFLOP/s (8.7k float atomics per 64 samples before), and
// the error against FP64 2.0e-6 to 2.8e-6 -> 0.1e-6 to 1.4e-6.
constexpr int GRAD_T = TSTRIDE * MT + MT * NF;  // transposition buffer of one wave, with the inputs
__global__ __launch_bounds__(64 * GRAD_WAVES) void k_mlp_grad(const float* __restrict__ params,
                                                              const float* __restrict__ X,
                                                              const float* __restrict__ T,
                                                              const uint32_t* __restrict__ perm, int64_t s0,
                                                              int64_t count, NormArgs nrm, float* __restrict__ part) {
    __shared__ __align__(16) float F[4 * FRAG], V[4 * NH], TB[GRAD_WAVES][GRAD_T];
    float *F2 = F, *F3 = F + FRAG, *B2 = F + 2 * FRAG, *B3 = F + 3 * FRAG;
    const int t = threadIdx.x, wave = t >> 6, lane = t & 63, g = lane >> 4, c = lane & 15;
    for (int e = t; e < FRAG; e += 64 * GRAD_WAVES) {
        const int at = frag_at(e / NH, e % NH), bt = frag_at(e % NH, e / NH);
        F2[at] = B2[bt] = params[OFF_W2 + e];
        F3[at] = B3[bt] = params[OFF_W3 + e];
    }
    for (int e = t; e < NH; e += 64 * GRAD_WAVES) {
        V[e] = params[OFF_B1 + e];
        V[NH + e] = params[OFF_B2 + e];
        V[2 * NH + e] = params[OFF_B3 + e];
        V[3 * NH + e] = params[OFF_W4 + e];
    }
    float w1[4];
#pragma unroll
    for (int o = 0; o < 4; o++) w1[o] = params[OFF_W1 + (16 * o + c) * NF + g];
    const float b4 = params[OFF_B4];
    const float xm = g == 0 ? nrm.xm[0] : g == 1 ? nrm.xm[1] : g == 2 ? nrm.xm[2] : nrm.xm[3];
    const float xs = g == 0 ? nrm.xs[0] : g == 1 ? nrm.xs[1] : g == 2 ? nrm.xs[2] : nrm.xs[3];
    __syncthreads();
    float* tb = TB[wave];
    float* tx = tb + TSTRIDE * MT;
    const f4 zero = {0.f, 0.f, 0.f, 0.f};
    f4 gw3[4][4], gw2[4][4], gw1[4], gw4[4];
    float gb3[4], gb2[4], gb4 = 0.f, loss = 0.f;
#pragma unroll
    for (int o = 0; o < 4; o++) {
#pragma unroll
        for (int i = 0; i < 4; i++) gw3[o][i] = gw2[o][i] = zero;
        gw1[o] = gw4[o] = zero;
        gb3[o] = gb2[o] = 0.f;
    }
    const int64_t tiles = (count + MT - 1) / MT, step = (int64_t)gridDim.x * GRAD_WAVES;
    int64_t tile = (int64_t)blockIdx.x * GRAD_WAVES + wave;
    // sample `at`: its feature and target, read one pass ahead
    float xn = 0.f, tn = 0.f;
    auto fetch = [&](int64_t at) {
        if (at < count) {
            int64_t idx = s0 + at;
            if (perm) idx = perm[idx];
            xn = X[idx * NF + g];
            tn = T[idx];
        }
    };
    fetch(tile * MT + c);
#pragma unroll 1
    for (; tile < tiles; tile += step) {
        const int64_t s = tile * MT + c;
        const bool live = s < count;
        const float x = live ? (xn - xm) / xs : 0.f;
        const float target = (tn - nrm.ym) / nrm.ys;
        fetch(s + step * MT);
        f4 h1[4], h2[4], z[4], p[4], q[4];
        const float y = mlp_layers(F2, F3, V, w1, b4, x, lane, h1, h2, z);
        const float d = live ? y - target : 0.f;
        gb4 += d;
        loss = __builtin_fmaf(0.5f * d, d, loss);
        const f4* w4 = (const f4*)V + 48 + g;
#pragma unroll
        for (int m = 0; m < 4; m++) {
            const f4 w = w4[m * 4];
#pragma unroll
            for (int r = 0; r < 4; r++) {
                gw4[m][r] = __builtin_fmaf(d, z[m][r], gw4[m][r]);
                z[m][r] = z[m][r] > 0.f ? d * w[r] : 0.f;
            }
        }
        // layer 3: its gradient, then back through its weights
        mlp_transpose(tb, lane, z, p);
        mlp_transpose(tb, lane, h2, q);
        mlp_outer(p, q, gw3);
#pragma unroll
        for (int m = 0; m < 4; m++) {
            gb3[m] += (p[m][0] + p[m][1]) + (p[m][2] + p[m][3]);
            q[m] = zero;
        }
        mlp_product(B3, lane, z, q);
#pragma unroll
        for (int m = 0; m < 4; m++)
#pragma unroll
            for (int r = 0; r < 4; r++) z[m][r] = h2[m][r] > 0.f ? q[m][r] : 0.f;
        // layer 2
        mlp_transpose(tb, lane, z, p);
        mlp_transpose(tb, lane, h1, q);
        mlp_outer(p, q, gw2);
#pragma unroll
        for (int m = 0; m < 4; m++) {
            gb2[m] += (p[m][0] + p[m][1]) + (p[m][2] + p[m][3]);
            q[m] = zero;
        }
        mlp_product(B2, lane, z, q);
#pragma unroll
        for (int m = 0; m < 4; m++)
#pragma unroll
            for (int r = 0; r < 4; r++) z[m][r] = h1[m][r] > 0.f ? q[m][r] : 0.f;
        // layer 1: columns 0-3 the inputs, column 4 the bias
        tx[c * NF + g] = x;
        mlp_transpose(tb, lane, z, p);
#pragma unroll
        for (int r = 0; r < 4; r++) {
            const float xr = c < NF ? tx[(4 * g + r) * NF + (c & (NF - 1))] : c == NF ? 1.f : 0.f;
#pragma unroll
            for (int o = 0; o < 4; o++) gw1[o] = __builtin_amdgcn_mfma_f32_16x16x4f32(p[o][r], xr, gw1[o], 0, 0, 0);
        }
        wave_fence();
    }
    // sums over the lanes that share an entry
    for (int k = 1; k < 16; k <<= 1) {
        gb4 += __shfl_xor(gb4, k);
        loss += __shfl_xor(loss, k);
#pragma unroll
        for (int m = 0; m < 4; m++)
#pragma unroll
            for (int r = 0; r < 4; r++) gw4[m][r] += __shfl_xor(gw4[m][r], k);
    }
#pragma unroll
    for (int m = 0; m < 4; m++) {
        gb3[m] += __shfl_xor(gb3[m], 16);
        gb3[m] += __shfl_xor(gb3[m], 32);
        gb2[m] += __shfl_xor(gb2[m], 16);
        gb2[m] += __shfl_xor(gb2[m], 32);
    }
    // the waves add their sums, one after the other, where the weights were
    float* G = F;
    for (int w = 0; w < GRAD_WAVES; w++) {
        __syncthreads();
        if (w != wave) continue;
        auto put = [&](int at, float v) { G[at] = w ? G[at] + v : v; };
#pragma unroll
        for (int o = 0; o < 4; o++)
#pragma unroll
            for (int r = 0; r < 4; r++) {
                const int u = 16 * o + 4 * g + r;
#pragma unroll
                for (int i = 0; i < 4; i++) {
                    put(OFF_W3 + u * NH + 16 * i + c, gw3[o][i][r]);
                    put(OFF_W2 + u * NH + 16 * i + c, gw2[o][i][r]);
                }
                if (c <= NF) put(c < NF ? OFF_W1 + u * NF + c : OFF_B1 + u, gw1[o][r]);
                if (c == 0) put(OFF_W4 + u, gw4[o][r]);
            }
        if (g == 0) {
#pragma unroll
            for (int m = 0; m < 4; m++) {
                put(OFF_B3 + 16 * m + c, gb3[m]);
                put(OFF_B2 + 16 * m + c, gb2[m]);
            }
        }
        if (lane == 0) {
            put(OFF_B4, gb4);
            put(NPARAM, loss);
        }
    }
    __syncthreads();
    float* out = part + (size_t)blockIdx.x * (NPARAM + 1);
    for (int e = t; e <= NPARAM; e += 64 * GRAD_WAVES) out[e] = G[e];
}

// grad = the sum of the workgroups' rows, in FP64: 32 entries a workgroup, 8
// threads on each
__global__ __launch_bounds__(256) void k_grad_sum(const float* __restrict__ part, int rows, float* __restrict__ grad) {
    __shared__ double S[8][32];
    const int c = threadIdx.x & 31, k = threadIdx.x >> 5, e = blockIdx.x * 32 + c;
    double v = 0.0;
    if (e <= NPARAM) {
#pragma unroll 8
        for (int r = k; r < rows; r += 8) v += (double)part[(size_t)r * (NPARAM + 1) + e];
    }
    S[k][c] = v;
    __syncthreads();
    if (k == 0 && e <= NPARAM) {
        for (int i = 1; i < 8; i++) v += S[i][c];
        grad[e] = (float)v;
    }
}

static void launch_forward(const float* params, const float* X, int64_t m, const NormArgs& n, float* Y,
                           hipStream_t st) {
    const int64_t b = (m + MT * FWD_WAVES - 1) / (MT * FWD_WAVES);
    hipLaunchKernelGGL(k_mlp_forward, dim3((unsigned)std::min<int64_t>(b, FWD_BLOCKS)), dim3(64 * FWD_WAVES), 0, st,
                       params, X, m, n, Y);
}

// gradient and loss of `count` samples into md->grad
static void launch_grad(const Model* md, const float* X, const float* T, const uint32_t* perm, int64_t s0,
                        int64_t count, const NormArgs& n, hipStream_t st) {
    const int64_t b = (count + MT * GRAD_WAVES - 1) / (MT * GRAD_WAVES);
    const int rows = (int)std::min<int64_t>(b, GRAD_BLOCKS);
    hipLaunchKernelGGL(k_mlp_grad, dim3(rows), dim3(64 * GRAD_WAVES), 0, st, md->params, X, T, perm, s0, count, n,
                       md->part);
    hipLaunchKernelGGL(k_grad_sum, dim3((NPARAM + 1 + 31) / 32), dim3(256), 0, st, (const float*)md->part, rows,
                       md->grad);
}

// Adam step on the gradient averaged over `count` samples.
__global__ void k_adam(float* __restrict__ params, const float* __restrict__ grad, float* __restrict__ m1,
                       float* __restrict__ m2, float inv_count, float lr, float b1, float b2, float eps, float c1,
                       float c2) {
    int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= NPARAM) return;
    const float g = grad[i] * inv_count;
    const float a = b1 * m1[i] + (1.f - b1) * g;
    const float v = b2 * m2[i] + (1.f - b2) * g * g;
    m1[i] = a;
    m2[i] = v;
    params[i] -= lr * (a / c1) / (sqrtf(v / c2) + eps);
}

// per-item features (log2(1 + A points), log2(1 + B points), transverse row
// separation in cells, cells per prune radius) and log2 of the recorded time
__global__ void k_item_features(const Item* __restrict__ items, const uint32_t* __restrict__ times, uint32_t n,
                                float kcells, float* __restrict__ X, float* __restrict__ logt) {
    uint32_t i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const Item it = items[i];
    const float na = (float)it.a_count;
    const float nb = (float)(it.b_end - it.b_begin);
    const float dy = (float)(int8_t)(it.meta & 0xffu), dz = (float)(int8_t)((it.meta >> 8) & 0xffu);
    X[4 * (size_t)i + 0] = log2f(1.f + na);
    X[4 * (size_t)i + 1] = log2f(1.f + nb);
    X[4 * (size_t)i + 2] = sqrtf(dy * dy + dz * dz);
    X[4 * (size_t)i + 3] = kcells;
    if (logt) logt[i] = log2f(1.f + (float)(times ? times[i] : 0u));
}

static void norm_args(const Model* md, NormArgs& n) {
    for (int i = 0; i < NF; i++) {
        n.xm[i] = md->norm[i];
        n.xs[i] = md->norm[NF + i];
    }
    n.ym = md->norm[8];
    n.ys = md->norm[9];
}

void model_item_costs(const Model* md, const Item* items, uint32_t n, float kcells, float* feat, float* pred,
                      hipStream_t st) {
    if (n == 0) return;
    NormArgs nrm;
    norm_args(md, nrm);
    hipLaunchKernelGGL(k_item_features, dim3((n + 255) / 256), dim3(256), 0, st, items, (const uint32_t*)nullptr, n,
                       kcells, feat, (float*)nullptr);
    launch_forward(md->params, feat, (int64_t)n, nrm, pred, st);
}

size_t model_param_bytes() { return sizeof(float) * (NPARAM + 1); }

Model* model_snapshot(const Model* src, float* params, hipStream_t st) {
    Model* m = new (std::nothrow) Model();
    if (!m) return nullptr;
    if (hipMemcpyAsync(params, src->params, model_param_bytes(), hipMemcpyDeviceToDevice, st) != hipSuccess) {
        delete m;
        return nullptr;
    }
    m->params = params;
    for (int i = 0; i < 10; i++) m->norm[i] = src->norm[i];
    m->step = src->step;
    return m;
}

void model_snapshot_free(Model* m) { delete m; }

static fcfc_status model_alloc(Model* md) {
    float* blk = nullptr;
    if (hipMalloc((void**)&blk, sizeof(float) * (4 * (NPARAM + 1) + 64)) != hipSuccess) {
        set_error("model: cannot allocate parameters");
        return FCFC_ENOMEM;
    }
    md->params = blk;
    md->grad = blk + (NPARAM + 1);
    md->m1 = blk + 2 * (NPARAM + 1);
    md->m2 = blk + 3 * (NPARAM + 1);
    FCFC_HIP(hipMemset(blk, 0, sizeof(float) * 4 * (NPARAM + 1)));
    return FCFC_OK;
}

// the workgroups' partial gradients, kept with the model
static fcfc_status model_partials(Model* md) {
    if (md->part) return FCFC_OK;
    if (hipMalloc((void**)&md->part, sizeof(float) * (size_t)GRAD_BLOCKS * (NPARAM + 1)) != hipSuccess) {
        md->part = nullptr;
        set_error("model: cannot allocate the partial gradients");
        return FCFC_ENOMEM;
    }
    return FCFC_OK;
}

}  // namespace fcfc

using namespace fcfc;

extern "C" int32_t fcfc_model_nparams(void) { return NPARAM; }

extern "C" fcfc_status fcfc_model_create(uint64_t seed, fcfc_model_t* out) {
    clear_error();
    if (!out) return FCFC_EINVAL;
    Model* md = new (std::nothrow) Model();
    if (!md) return FCFC_ENOMEM;
    fcfc_status s = model_alloc(md);
    if (s != FCFC_OK) {
        delete md;
        return s;
    }
    // He-uniform initialisation (host, seeded)
    std::vector<float> h(NPARAM, 0.f);
    std::mt19937_64 rng(seed);
    auto fill = [&](int off, int nout, int nin) {
        float lim = sqrtf(6.f / (float)nin);
        std::uniform_real_distribution<float> u(-lim, lim);
        for (int i = 0; i < nout * nin; i++) h[off + i] = u(rng);
    };
    fill(OFF_W1, NH, NF);
    fill(OFF_W2, NH, NH);
    fill(OFF_W3, NH, NH);
    fill(OFF_W4, 1, NH);
    FCFC_HIP(hipMemcpy(md->params, h.data(), sizeof(float) * NPARAM, hipMemcpyHostToDevice));
    *out = (fcfc_model_t)md;
    return FCFC_OK;
}

extern "C" void fcfc_model_free(fcfc_model_t model) {
    Model* md = (Model*)model;
    if (!md) return;
    if (md->params) (void)hipFree(md->params);
    if (md->part) (void)hipFree(md->part);
    delete md;
}

extern "C" fcfc_status fcfc_model_get(fcfc_model_t model, float* params, float* norm) {
    Model* md = (Model*)model;
    if (!md) return FCFC_EINVAL;
    if (params) FCFC_HIP(hipMemcpy(params, md->params, sizeof(float) * NPARAM, hipMemcpyDeviceToHost));
    if (norm) memcpy(norm, md->norm, sizeof(md->norm));
    return FCFC_OK;
}

extern "C" fcfc_status fcfc_model_set(fcfc_model_t model, const float* params, const float* norm) {
    Model* md = (Model*)model;
    if (!md) return FCFC_EINVAL;
    if (params) FCFC_HIP(hipMemcpy(md->params, params, sizeof(float) * NPARAM, hipMemcpyHostToDevice));
    if (norm) {
        for (int i = 0; i < 10; i++)
            if (!isfinite(norm[i]) || (i >= NF && i < 2 * NF && !(norm[i] > 0)) || (i == 9 && !(norm[i] > 0))) {
                set_error("model_set: normalisation must be finite with positive scales");
                return FCFC_EINVAL;
            }
        memcpy(md->norm, norm, sizeof(md->norm));
    }
    md->step = 0;
    FCFC_HIP(hipMemset(md->m1, 0, sizeof(float) * 2 * (NPARAM + 1)));
    return FCFC_OK;
}

extern "C" fcfc_status fcfc_model_predict(fcfc_model_t model, const float* d_feat, int64_t m, float* d_out,
                                          void* stream) {
    clear_error();
    Model* md = (Model*)model;
    if (!md || (m > 0 && (!d_feat || !d_out)) || m < 0) return FCFC_EINVAL;
    if (m == 0) return FCFC_OK;
    NormArgs n;
    norm_args(md, n);
    launch_forward(md->params, d_feat, m, n, d_out, (hipStream_t)stream);
    FCFC_HIP(hipGetLastError());
    return FCFC_OK;
}

extern "C" fcfc_status fcfc_model_grad(fcfc_model_t model, const float* d_feat, const float* d_target, int64_t m,
                                       float* grad_host, float* loss_host, void* stream) {
    clear_error();
    Model* md = (Model*)model;
    if (!md || m <= 0 || !d_feat || !d_target) return FCFC_EINVAL;
    hipStream_t st = (hipStream_t)stream;
    NormArgs n;
    norm_args(md, n);
    FCFC_TRY(model_partials(md));
    launch_grad(md, d_feat, d_target, nullptr, 0, m, n, st);
    FCFC_HIP(hipGetLastError());
    std::vector<float> h(NPARAM + 1);
    FCFC_HIP(hipMemcpyAsync(h.data(), md->grad, sizeof(float) * (NPARAM + 1), hipMemcpyDeviceToHost, st));
    FCFC_HIP(hipStreamSynchronize(st));
    if (grad_host) memcpy(grad_host, h.data(), sizeof(float) * NPARAM);
    if (loss_host) *loss_host = h[NPARAM];
    return FCFC_OK;
}

// Standardisation from the training set (host copies), then `epochs` passes of
// Adam over shuffled minibatches of `batch` samples.  Returns the mean loss of
// the last epoch (standardised units).
extern "C" fcfc_status fcfc_model_train(fcfc_model_t model, const float* d_feat, const float* d_target, int64_t m,
                                        int32_t epochs, int32_t batch, float lr, uint64_t seed, void* stream,
                                        float* final_loss) {
    clear_error();
    Model* md = (Model*)model;
    if (!md || m < 2 || !d_feat || !d_target || epochs < 1 || batch < MB || !(lr > 0)) {
        set_error("model_train: need m >= 2 samples, epochs >= 1, batch >= %d, lr > 0", MB);
        return FCFC_EINVAL;
    }
    hipStream_t st = (hipStream_t)stream;
    std::vector<float> hx((size_t)m * NF), ht((size_t)m);
    FCFC_HIP(hipMemcpyAsync(hx.data(), d_feat, hx.size() * 4, hipMemcpyDeviceToHost, st));
    FCFC_HIP(hipMemcpyAsync(ht.data(), d_target, ht.size() * 4, hipMemcpyDeviceToHost, st));
    FCFC_HIP(hipStreamSynchronize(st));
    for (int f = 0; f < NF; f++) {
        double s = 0, s2 = 0;
        for (int64_t i = 0; i < m; i++) {
            double v = hx[i * NF + f];
            s += v;
            s2 += v * v;
        }
        double mu = s / m, var = s2 / m - mu * mu;
        md->norm[f] = (float)mu;
        md->norm[NF + f] = (float)std::max(sqrt(std::max(var, 0.0)), 1e-3);
    }
    {
        double s = 0, s2 = 0;
        for (int64_t i = 0; i < m; i++) {
            s += ht[i];
            s2 += (double)ht[i] * ht[i];
        }
        double mu = s / m, var = s2 / m - mu * mu;
        md->norm[8] = (float)mu;
        md->norm[9] = (float)std::max(sqrt(std::max(var, 0.0)), 1e-3);
    }
    NormArgs n;
    norm_args(md, n);
    FCFC_TRY(model_partials(md));
    uint32_t* perm = nullptr;
    FCFC_HIP(hipMalloc((void**)&perm, sizeof(uint32_t) * (size_t)m));
    std::vector<uint32_t> hp((size_t)m);
    for (int64_t i = 0; i < m; i++) hp[i] = (uint32_t)i;
    std::mt19937_64 rng(seed);
    float last = 0.f;
    const float b1 = 0.9f, b2 = 0.999f, eps = 1e-8f;
    for (int e = 0; e < epochs; e++) {
        std::shuffle(hp.begin(), hp.end(), rng);
        FCFC_HIP(hipMemcpyAsync(perm, hp.data(), sizeof(uint32_t) * (size_t)m, hipMemcpyHostToDevice, st));
        double eloss = 0;
        for (int64_t s0 = 0; s0 < m; s0 += batch) {
            const int64_t cnt = std::min<int64_t>(batch, m - s0);
            launch_grad(md, d_feat, d_target, perm, s0, cnt, n, st);
            md->step++;
            const float c1 = 1.f - powf(b1, (float)md->step), c2 = 1.f - powf(b2, (float)md->step);
            if (e == epochs - 1) {
                float l = 0.f;
                FCFC_HIP(hipMemcpyAsync(&l, md->grad + NPARAM, 4, hipMemcpyDeviceToHost, st));
                FCFC_HIP(hipStreamSynchronize(st));
                eloss += l;
            }
            hipLaunchKernelGGL(k_adam, dim3((NPARAM + 256) / 256), dim3(256), 0, st, md->params, md->grad, md->m1, md->m2,
                               1.f / (float)cnt, lr, b1, b2, eps, c1, c2);
        }
        if (e == epochs - 1) last = (float)(eloss / m);
    }
    FCFC_HIP(hipStreamSynchronize(st));
    (void)hipFree(perm);
    if (final_loss) *final_loss = last;
    return FCFC_OK;
}

extern "C" fcfc_status fcfc_model_save(fcfc_model_t model, const char* path) {
    clear_error();
    Model* md = (Model*)model;
    if (!md || !path) return FCFC_EINVAL;
    std::vector<float> h(NPARAM);
    FCFC_HIP(hipMemcpy(h.data(), md->params, sizeof(float) * NPARAM, hipMemcpyDeviceToHost));
    FILE* f = fopen(path, "wb");
    if (!f) {
        set_error("model_save: cannot open %s", path);
        return FCFC_EINVAL;
    }
    const char magic[8] = {'F', 'C', 'F', 'C', 'M', 'L', 'P', '1'};
    int32_t np = NPARAM;
    bool ok = fwrite(magic, 1, 8, f) == 8 && fwrite(&np, 4, 1, f) == 1 && fwrite(md->norm, 4, 10, f) == 10 &&
              fwrite(h.data(), 4, NPARAM, f) == (size_t)NPARAM;
    fclose(f);
    if (!ok) {
        set_error("model_save: write failed");
        return FCFC_EINVAL;
    }
    return FCFC_OK;
}

extern "C" fcfc_status fcfc_model_load(const char* path, fcfc_model_t* out) {
    clear_error();
    if (!path || !out) return FCFC_EINVAL;
    FILE* f = fopen(path, "rb");
    if (!f) {
        set_error("model_load: cannot open %s", path);
        return FCFC_EMODEL;
    }
    char magic[8];
    int32_t np = 0;
    float norm[10];
    std::vector<float> h(NPARAM);
    bool ok = fread(magic, 1, 8, f) == 8 && memcmp(magic, "FCFCMLP1", 8) == 0 && fread(&np, 4, 1, f) == 1 &&
              np == NPARAM && fread(norm, 4, 10, f) == 10 && fread(h.data(), 4, NPARAM, f) == (size_t)NPARAM;
    fclose(f);
    for (int i = 0; ok && i < NPARAM; i++) ok = isfinite(h[i]);
    if (!ok) {
        set_error("model_load: %s is not a valid model file", path);
        return FCFC_EMODEL;
    }
    fcfc_model_t m = nullptr;
    FCFC_TRY(fcfc_model_create(0, &m));
    fcfc_status s = fcfc_model_set(m, h.data(), norm);
    if (s != FCFC_OK) {
        fcfc_model_free(m);
        set_error("model_load: invalid normalisation in %s", path);
        return FCFC_EMODEL;
    }
    *out = m;
    return FCFC_OK;
}

// Features (and log2 time) of the work items of the last count recorded with
// record_timing = 1 on this plan.  d_feat: cap x 4 floats, d_logt: cap floats.
extern "C" fcfc_status fcfc_plan_timings(fcfc_plan_t plan, float* d_feat, float* d_logt, int64_t cap, int64_t* n,
                                         void* stream) {
    clear_error();
    Plan* p = (Plan*)plan;
    if (!p || !n) return FCFC_EINVAL;
    if (!p->timing_dev || p->timing_n == 0) {
        set_error("plan_timings: no count with record_timing = 1 has run on this plan");
        return FCFC_ESTATE;
    }
    *n = p->timing_n;
    if (!d_feat) return FCFC_OK;
    if (cap < (int64_t)p->timing_n) {
        set_error("plan_timings: capacity %lld < %u items", (long long)cap, p->timing_n);
        return FCFC_EINVAL;
    }
    const uint32_t* times = (const uint32_t*)p->timing_dev;
    const Item* items = (const Item*)((const char*)p->timing_dev + (size_t)p->timing_n * 4);
    const float kc = (float)(p->rprune / p->grid.side);
    hipLaunchKernelGGL(k_item_features, dim3((p->timing_n + 255) / 256), dim3(256), 0, (hipStream_t)stream, items,
                       times, p->timing_n, kc, d_feat, d_logt);
    FCFC_HIP(hipGetLastError());
    return FCFC_OK;
}

extern "C" fcfc_status fcfc_plan_set_model(fcfc_plan_t plan, fcfc_model_t model) {
    clear_error();
    Plan* p = (Plan*)plan;
    if (!p) return FCFC_EINVAL;
    p->model = (Model*)model;
    return FCFC_OK;
}

extern "C" fcfc_status fcfc_plan_predict(fcfc_plan_t plan, fcfc_cells_t c1, fcfc_cells_t c2, fcfc_model_t model,
                                         void* stream, double* pred_ms, int64_t* n_items) {
    clear_error();
    Plan* p = (Plan*)plan;
    Cells* a = (Cells*)c1;
    Cells* b = (Cells*)c2;
    if (!p || !a || !model || !pred_ms) {
        set_error("plan_predict: null plan, cells, model or output");
        return FCFC_EINVAL;
    }
    if (a->plan_id != p->id || (b && b->plan_id != p->id)) {
        set_error("plan_predict: cell sets were built on a different plan");
        return FCFC_EGRID;
    }
    PredictReq pr;
    pr.model = (const Model*)model;
    FCFC_TRY(count_pairs(p, a, b, nullptr, nullptr, (hipStream_t)stream, &pr));
    *pred_ms = pr.pred_ms;
    if (n_items) *n_items = pr.items;
    return FCFC_OK;
}

extern "C" fcfc_status fcfc_choose_cells(fcfc_model_t model, int32_t kind, int32_t los, const double* edges1,
                                         int32_t n1, const double* edges2, int32_t n2, double box_L,
                                         const fcfc_tuning* tune, const fcfc_catalog* c1, const fcfc_catalog* c2,
                                         void* stream, int32_t* best_k, double pred_ms[6]) {
    clear_error();
    if (!c1 || !best_k) {
        set_error("choose_cells: null catalogue or output");
        return FCFC_EINVAL;
    }
    fcfc_tuning t{};
    if (tune) t = *tune;
    if (t.n_hint <= 0) t.n_hint = (int32_t)std::min<int64_t>(c1->n, 0x7fffffff);
    t.record_timing = 0;
    for (int k = 0; k < 6; k++)
        if (pred_ms) pred_ms[k] = NAN;
    const fcfc_catalog a{c1->xyz, nullptr, c1->n};
    const fcfc_catalog b{c2 ? c2->xyz : nullptr, nullptr, c2 ? c2->n : 0};
    fcfc_catalog both[2] = {a, b};
    auto make = [&](int k, fcfc_plan_t* pl) -> fcfc_status {
        t.cells_per_rmax = k;
        FCFC_TRY(fcfc_plan_create(kind, los, edges1, n1, edges2, n2, box_L, &t, pl));
        if (box_L <= 0) {
            fcfc_status s = fcfc_plan_fit_bounds(*pl, both, c2 ? 2 : 1, stream);
            if (s != FCFC_OK) {
                fcfc_plan_free(*pl);
                return s;
            }
        }
        return FCFC_OK;
    };
    if (!model) {
        fcfc_plan_t pl = nullptr;
        FCFC_TRY(make(tune ? tune->cells_per_rmax : 0, &pl));
        *best_k = ((Plan*)pl)->grid.k;
        fcfc_plan_free(pl);
        return FCFC_OK;
    }
    double best = INFINITY;
    int bk = 0;
    for (int k = 1; k <= 6; k++) {
        fcfc_plan_t pl = nullptr;
        fcfc_status s = make(k, &pl);
        if (s == FCFC_ERANGE) continue;  // grid too fine for this box
        FCFC_TRY(s);
        if (((Plan*)pl)->grid.k != k) {
            fcfc_plan_free(pl);
            continue;
        }
        fcfc_cells_t ca = nullptr, cb = nullptr;
        s = fcfc_build_cells(pl, &a, stream, &ca);
        if (s == FCFC_OK && c2) s = fcfc_build_cells(pl, &b, stream, &cb);
        double ms = NAN;
        if (s == FCFC_OK) s = fcfc_plan_predict(pl, ca, cb, model, stream, &ms, nullptr);
        fcfc_cells_free(ca);
        fcfc_cells_free(cb);
        fcfc_plan_free(pl);
        FCFC_TRY(s);
        if (pred_ms) pred_ms[k - 1] = ms;
        if (isfinite(ms) && ms < best) {
            best = ms;
            bk = k;
        }
    }
    if (bk == 0) {
        // no usable prediction: the analytic choice
        fcfc_plan_t pl = nullptr;
        FCFC_TRY(make(0, &pl));
        bk = ((Plan*)pl)->grid.k;
        fcfc_plan_free(pl);
    }
    *best_k = bk;
    return FCFC_OK;
}
