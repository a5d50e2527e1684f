// Learned subgrid closure: parameters, GPU training kernels (FP32 master
// weights, forward, backward, Adam) and BF16 matrix-core inference.
//
// Parameter order (float32, 5254 values): W1[10][64], b1[64], W2[64][64],
// b2[64], W3[64][6], b3[6]; a layer computes h_out = h_in W + b.  Loss:
// L = (1/N) sum_n sum_c w_c (z_nc - t_nc)^2 with z = y minus the trace of its
// (xx, yy, zz) part and w = (1, 1, 1, 2, 2, 2) (Frobenius norm of the
// symmetric tensor).  Adam: bias-corrected moments, beta1 0.9, beta2 0.999,
// eps 1e-8.  Every reduction over samples runs in a fixed order.
#include <algorithm>
#include <cmath>
#include <cstring>
#include <mutex>
#include <string>

#include "mlp.hpp"

namespace lesasm {

constexpr int OFF_W1 = 0, OFF_B1 = OFF_W1 + kMlpIn * kMlpH, OFF_W2 = OFF_B1 + kMlpH, OFF_B2 = OFF_W2 + kMlpH * kMlpH,
              OFF_W3 = OFF_B2 + kMlpH, OFF_B3 = OFF_W3 + kMlpH * kMlpOut;

// ---- FP32 matrix-core forward and training ------------------------------------
//
// v_mfma_f32_16x16x4_f32 (FP32 operands and sums):
//   A[i][k] in lane i + 16 k,  B[k][j] in lane j + 16 k,  D[i][j] in lane j + 16 (i/4), slot i%4.
// A wavefront carries 16 samples through the network transposed, H^T = W^T
// X^T: lane j + 16 q then holds, of sample j, units 16 m + 4 q + r in slot r
// of row tile m.  Used slot by slot as the B operand of the next product, slot
// r supplies units {4 q + r}, so numbering the K index of the weights the same
// way chains the layers, forward and backward, with no movement between lanes.
struct NetLds {
    // Rows of 68 floats: 16 rows (or 4 rows of 4 groups) then fall on different
    // banks, and 4 consecutive units are one aligned 16-byte read.
    float w1[12][68];       // W1[10][64], row 10 = b1 (input 10 is the constant 1), row 11 = 0
    float w2[kMlpH][68];    // W2[64][64]
    float w3[kMlpH][8];     // W3[64][6], columns 6 and 7 = 0
    float b2[kMlpH], b3[16];
};

// Copies the parameters into LDS; call with the whole workgroup, then a barrier.
__device__ __forceinline__ void net_stage(const float *__restrict__ P, NetLds &w) {
    for (int k = threadIdx.x; k < 12 * kMlpH; k += blockDim.x)
        w.w1[k / kMlpH][k % kMlpH] = k < 11 * kMlpH ? P[OFF_W1 + k] : 0.f;  // b1 follows W1
    for (int k = threadIdx.x; k < kMlpH * kMlpH; k += blockDim.x) w.w2[k / kMlpH][k % kMlpH] = P[OFF_W2 + k];
    for (int k = threadIdx.x; k < kMlpH * 8; k += blockDim.x)
        w.w3[k / 8][k % 8] = k % 8 < kMlpOut ? P[OFF_W3 + (k / 8) * kMlpOut + k % 8] : 0.f;
    for (int k = threadIdx.x; k < kMlpH; k += blockDim.x) w.b2[k] = P[OFF_B2 + k];
    if (threadIdx.x < 16) w.b3[threadIdx.x] = threadIdx.x < kMlpOut ? P[OFF_B3 + threadIdx.x] : 0.f;
}
static_assert(OFF_B1 == OFF_W1 + kMlpIn * kMlpH, "b1 follows W1");

__device__ __forceinline__ f32x4_t relu4(f32x4_t v) {
#pragma unroll
    for (int r = 0; r < 4; ++r) v[r] = v[r] > 0.f ? v[r] : 0.f;
    return v;
}

// Inputs of sample s (lane j + 16 q: features 4 t + q), the constant 1 as
// feature 10; a sample past the end has zeros, the constant included.
__device__ __forceinline__ void net_inputs(const float *__restrict__ X, int64_t s, int n, int q, float (&x)[3]) {
#pragma unroll
    for (int t = 0; t < 3; ++t) {
        const int f = 4 * t + q;
        x[t] = s >= n || f > kMlpIn ? 0.f : f == kMlpIn ? 1.f : X[s * kMlpIn + f];
    }
}

// Both hidden layers (after ReLU) and the outputs (rows 0-5 of the tile) of 16 samples.
__device__ __forceinline__ void net_forward(const NetLds &w, int c, int q, const float (&x)[3], f32x4_t (&h1)[4],
                                            f32x4_t (&h2)[4], f32x4_t &y) {
#pragma unroll
    for (int m = 0; m < 4; ++m) h1[m] = f32x4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int t = 0; t < 3; ++t)
#pragma unroll
        for (int m = 0; m < 4; ++m)
            h1[m] = __builtin_amdgcn_mfma_f32_16x16x4f32(w.w1[4 * t + q][16 * m + c], x[t], h1[m], 0, 0, 0);
#pragma unroll
    for (int m = 0; m < 4; ++m) {
        h1[m] = relu4(h1[m]);
        h2[m] = *(const f32x4_t *)&w.b2[16 * m + 4 * q];
    }
#pragma unroll
    for (int t = 0; t < 4; ++t)
#pragma unroll
        for (int r = 0; r < 4; ++r)
#pragma unroll
            for (int m = 0; m < 4; ++m)
                h2[m] = __builtin_amdgcn_mfma_f32_16x16x4f32(w.w2[16 * t + 4 * q + r][16 * m + c], h1[t][r], h2[m], 0, 0, 0);
#pragma unroll
    for (int m = 0; m < 4; ++m) h2[m] = relu4(h2[m]);
    y = *(const f32x4_t *)&w.b3[4 * q];
    f32x4_t y1 = {0.f, 0.f, 0.f, 0.f};  // two chains of half the length
#pragma unroll
    for (int t = 0; t < 4; t += 2)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const float a0 = w.w3[16 * t + 4 * q + r][c & 7], a1 = w.w3[16 * t + 16 + 4 * q + r][c & 7];
            y = __builtin_amdgcn_mfma_f32_16x16x4f32(c < 8 ? a0 : 0.f, h2[t][r], y, 0, 0, 0);
            y1 = __builtin_amdgcn_mfma_f32_16x16x4f32(c < 8 ? a1 : 0.f, h2[t + 1][r], y1, 0, 0, 0);
        }
    y += y1;
}

// Loss and weight gradients of n samples.  A workgroup takes tiles of 64
// samples (tile b, b + grid, ...): each wavefront runs its 16 samples forward
// and back in registers and leaves inputs, activations and their gradients in
// LDS; then the four wavefronts share the weight gradients (K = the 64
// samples), which stay in accumulators over the workgroup's tiles.  The sums of
// one workgroup go to partial[b] (the parameters' order, then the loss), and
// k_mlp_grad_reduce adds the workgroups in a fixed order.
// Bound by latency, not by bytes (64 B a sample): of 17 us with one tile a
// workgroup the 268 FP32 matrix instructions of a wavefront take 3.6 (32 cycles
// each), the rest is the parameters' and samples' way into LDS and the layers'
// dependences (waiting 0.60 of the wave time).  The kernels
// it replaces kept H1, H2 and their gradients in memory (1052 B a sample) and
// summed each weight's gradient over all samples in one thread: loss and
// gradients of 8192 samples 17 against 2064 us (call to call, host included),
// of a million 0.47 against 333 ms; forward_f32 of a million 107 against 327 us.
constexpr int kTrainTile = 64;
constexpr int kTrainMaxBlocks = 256;           // one per compute unit (98 KB of LDS each)
constexpr int kPartialStride = kMlpParams + 2;  // the loss at kMlpParams
struct TrainLds {
    NetLds w;
    float h1[kTrainTile][68], h2[kTrainTile][68], da1[kTrainTile][68], da2[kTrainTile][68];
    float x[kTrainTile][20], dy[kTrainTile][12];
    float loss[4];
};

inline int train_blocks(int n) { return std::min((n - 1) / kTrainTile + 1, kTrainMaxBlocks); }

__global__ __launch_bounds__(256) void k_mlp_train(const float *__restrict__ P, const float *__restrict__ X,
                                                   const float *__restrict__ Tg, int n, float *__restrict__ partial) {
    extern __shared__ __align__(16) unsigned char smem[];
    TrainLds &L = *(TrainLds *)smem;
    net_stage(P, L.w);
    __syncthreads();
    const int wave = threadIdx.x / 64, lane = threadIdx.x % 64, c = lane & 15, q = lane >> 4;
    const f32x4_t zero = {0.f, 0.f, 0.f, 0.f};
    f32x4_t g1 = zero, g2[4] = {zero, zero, zero, zero}, g3 = zero;
    float gb2 = 0.f, gb3 = 0.f, loss = 0.f;
    const int ntiles = (n - 1) / kTrainTile + 1;
    for (int tile = blockIdx.x; tile < ntiles; tile += gridDim.x) {
        const int sl = 16 * wave + c;
        const int64_t s = (int64_t)tile * kTrainTile + sl;
        float x[3];
        net_inputs(X, s, n, q, x);
        f32x4_t h1[4], h2[4], y;
        net_forward(L.w, c, q, x, h1, h2, y);
        // the sums over the tile run over samples past the end too: theirs are zero
        // (h1 is, by its inputs; h2 would hold b2, and a gradient of zero times an
        // infinity is not zero)
        if (s >= n) h2[0] = h2[1] = h2[2] = h2[3] = zero;
        // loss term and dL/dy through the trace projection: lane group 0 holds
        // components 0-3, group 1 components 4 and 5
        if (q == 0) {
            const float tr = (y[0] + y[1] + y[2]) * (1.0f / 3.0f);
            y[0] -= tr;
            y[1] -= tr;
            y[2] -= tr;
        }
        f32x4_t dy = zero;
        float l = 0.f;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int o = 4 * q + r;
            if (o < kMlpOut && s < n) {
                const float wt = o < 3 ? 1.f : 2.f, d = y[r] - Tg[s * kMlpOut + o];
                l += wt * d * d;
                dy[r] = 2.f * wt * d / (float)n;
            }
        }
        loss += l / (float)n;
        if (q == 0) {
            const float m = (dy[0] + dy[1] + dy[2]) * (1.0f / 3.0f);
            dy[0] -= m;
            dy[1] -= m;
            dy[2] -= m;
        }
        f32x4_t da1[4], da2[4];
#pragma unroll
        for (int m = 0; m < 4; ++m) {
            const f32x4_t a = *(const f32x4_t *)&L.w.w3[16 * m + c][4 * (q & 1)];
            da2[m] = zero;
#pragma unroll
            for (int r = 0; r < 4; ++r)
                da2[m] = __builtin_amdgcn_mfma_f32_16x16x4f32(q < 2 ? a[r] : 0.f, dy[r], da2[m], 0, 0, 0);
#pragma unroll
            for (int r = 0; r < 4; ++r) da2[m][r] = h2[m][r] > 0.f ? da2[m][r] : 0.f;
            da1[m] = zero;
        }
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            f32x4_t a[4];
#pragma unroll
            for (int m = 0; m < 4; ++m) a[m] = *(const f32x4_t *)&L.w.w2[16 * m + c][16 * t + 4 * q];
#pragma unroll
            for (int r = 0; r < 4; ++r)
#pragma unroll
                for (int m = 0; m < 4; ++m)
                    da1[m] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[m][r], da2[t][r], da1[m], 0, 0, 0);
        }
#pragma unroll
        for (int m = 0; m < 4; ++m) {
#pragma unroll
            for (int r = 0; r < 4; ++r) da1[m][r] = h1[m][r] > 0.f ? da1[m][r] : 0.f;
            *(f32x4_t *)&L.h1[sl][16 * m + 4 * q] = h1[m];
            *(f32x4_t *)&L.h2[sl][16 * m + 4 * q] = h2[m];
            *(f32x4_t *)&L.da1[sl][16 * m + 4 * q] = da1[m];
            *(f32x4_t *)&L.da2[sl][16 * m + 4 * q] = da2[m];
        }
#pragma unroll
        for (int t = 0; t < 3; ++t) L.x[sl][4 * t + q] = x[t];
        L.x[sl][12 + q] = 0.f;
        if (q < 2) *(f32x4_t *)&L.dy[sl][4 * q] = dy;
        __syncthreads();
        // weight gradients: wavefront w takes columns 16 w .. 16 w + 15 of W1
        // (with b1) and W2 and rows 16 w .. of W3; A[unit][sample], B[sample][unit]
#pragma unroll 4
        for (int t = 0; t < kTrainTile / 4; ++t) {
            const int k = 4 * t + q;
            const float b1 = L.da1[k][16 * wave + c], b2 = L.da2[k][16 * wave + c];
            const float b3 = c < 8 ? L.dy[k][c & 7] : 0.f;
            g1 = __builtin_amdgcn_mfma_f32_16x16x4f32(L.x[k][c], b1, g1, 0, 0, 0);
#pragma unroll
            for (int m = 0; m < 4; ++m)
                g2[m] = __builtin_amdgcn_mfma_f32_16x16x4f32(L.h1[k][16 * m + c], b2, g2[m], 0, 0, 0);
            g3 = __builtin_amdgcn_mfma_f32_16x16x4f32(L.h2[k][16 * wave + c], b3, g3, 0, 0, 0);
            gb2 += b2;
            gb3 += b3;
        }
        __syncthreads();  // the next tile overwrites the LDS
    }
    float *out = partial + (size_t)blockIdx.x * kPartialStride;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const int i = 4 * q + r;
        if (i <= kMlpIn) out[OFF_W1 + i * kMlpH + 16 * wave + c] = g1[r];  // row 10: b1
#pragma unroll
        for (int m = 0; m < 4; ++m) out[OFF_W2 + (16 * m + i) * kMlpH + 16 * wave + c] = g2[m][r];
        if (c < kMlpOut) out[OFF_W3 + (16 * wave + i) * kMlpOut + c] = g3[r];
    }
    gb2 += __shfl_xor(gb2, 16);
    gb2 += __shfl_xor(gb2, 32);
    gb3 += __shfl_xor(gb3, 16);
    gb3 += __shfl_xor(gb3, 32);
    if (q == 0) out[OFF_B2 + 16 * wave + c] = gb2;
    if (wave == 0 && q == 0 && c < kMlpOut) out[OFF_B3 + c] = gb3;
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) loss += __shfl_xor(loss, o);
    if (lane == 0) L.loss[wave] = loss;
    __syncthreads();
    if (threadIdx.x == 0) out[kMlpParams] = (L.loss[0] + L.loss[1]) + (L.loss[2] + L.loss[3]);
}

// grad[j] (and *loss, if wanted) = sum over the workgroups' partial sums, in a
// fixed order: 8 interleaved slices of the workgroups, then the slices.
__global__ __launch_bounds__(512) void k_mlp_grad_reduce(const float *__restrict__ partial, int nb,
                                                         float *__restrict__ grad, float *__restrict__ loss) {
    __shared__ float sh[8][64];
    const int l = threadIdx.x & 63, slice = threadIdx.x >> 6, j = blockIdx.x * 64 + l;
    float s = 0.f;
    if (j <= kMlpParams)
#pragma unroll 8
        for (int b = slice; b < nb; b += 8) s += partial[(size_t)b * kPartialStride + j];
    sh[slice][l] = s;
    __syncthreads();
    if (slice != 0 || j > kMlpParams) return;
    s = 0.f;
#pragma unroll
    for (int k = 0; k < 8; ++k) s += sh[k][l];
    if (j < kMlpParams)
        grad[j] = s;
    else if (loss)
        *loss = s;
}

__global__ void k_adam(float *__restrict__ P, float *__restrict__ M, float *__restrict__ V,
                       const float *__restrict__ g, int n, float lr, float c1, float c2) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const float gi = g[i];
    const float m = 0.9f * M[i] + 0.1f * gi;
    const float v = 0.999f * V[i] + 0.001f * gi * gi;
    M[i] = m;
    V[i] = v;
    P[i] -= lr * (m / c1) / (sqrtf(v / c2) + 1e-8f);
}

// FP32 outputs of n samples: 16 samples per wavefront and round, bound by the
// FP32 matrix instructions (92 of 32 cycles per 16 samples).
__global__ __launch_bounds__(256) void k_mlp_forward_f32(const float *__restrict__ P, const float *__restrict__ X,
                                                         int n, float *__restrict__ Y) {
    __shared__ __align__(16) NetLds w;
    net_stage(P, w);
    __syncthreads();
    const int wave = threadIdx.x / 64, lane = threadIdx.x % 64, c = lane & 15, q = lane >> 4;
    for (int64_t base = (blockIdx.x * 4 + wave) * 16; base < n; base += gridDim.x * 64) {
        const int64_t s = base + c;
        float x[3];
        net_inputs(X, s, n, q, x);
        f32x4_t h1[4], h2[4], y;
        net_forward(w, c, q, x, h1, h2, y);
#pragma unroll
        for (int r = 0; r < 4; ++r)
            if (s < n && 4 * q + r < kMlpOut) Y[s * kMlpOut + 4 * q + r] = y[r];
    }
}

// Matrix-core inference of N samples: each wavefront takes 64 samples at a
// time (the last group padded by repeating the final sample).
__global__ __launch_bounds__(256) void k_mlp_infer_bf16(const short *__restrict__ packed,
                                                        const float *__restrict__ bias, const float *__restrict__ X,
                                                        int n, float *__restrict__ Y) {
    extern __shared__ __align__(16) unsigned char smem[];
    const MlpLds w = mlp_stage(packed, bias, smem);
    __syncthreads();
    const int wave = threadIdx.x / 64, lane = threadIdx.x % 64;
    unsigned char *scratch = smem + kMlpLdsBytes + wave * kMlpWaveScratch;
    const int waves = gridDim.x * (blockDim.x / 64);
    for (int base = (blockIdx.x * (blockDim.x / 64) + wave) * 64; base < n; base += waves * 64) {
        const int i = min(base + lane, n - 1);
        float x[kMlpIn], y[kMlpOut];
        for (int k = 0; k < kMlpIn; ++k) x[k] = X[(size_t)i * kMlpIn + k];
        mlp_wave(w, x, y, scratch);
        if (base + lane < n)
            for (int o = 0; o < kMlpOut; ++o) Y[(size_t)i * kMlpOut + o] = y[o];
    }
}

// Packs float parameters into the A tiles of mlp_wave (bf16) and the bias block.
static void pack_weights(const float *P, std::vector<short> &tiles, std::vector<float> &bias) {
    auto bf = [](float f) -> short {
        uint32_t u;
        std::memcpy(&u, &f, 4);
        u += 0x7FFFu + ((u >> 16) & 1u);
        return (short)(u >> 16);
    };
    tiles.assign(kMlpPackedShorts, 0);
    auto put = [&](int tile, int i, int k, float v) {  // A[i][k] of a 16x16 tile
        const int lane = i + 16 * (k / 4);
        tiles[((size_t)tile * 64 + lane) * 4 + (k % 4)] = bf(v);
    };
    for (int mt = 0; mt < 4; ++mt)  // W1^T: rows = hidden, k = input
        for (int i = 0; i < 16; ++i)
            for (int k = 0; k < 16; ++k) put(mt, i, k, k < kMlpIn ? P[OFF_W1 + k * kMlpH + 16 * mt + i] : 0.f);
    // W2^T tiles (mt, kb) of K = 32: A[i][k] in lane i + 16 (k/8), slot k%8;
    // K index k of block kb is hidden unit 16 (2 kb + s/4) + 4 (k/8) + s%4, s = k%8
    for (int mt = 0; mt < 4; ++mt)
        for (int kb = 0; kb < 2; ++kb)
            for (int i = 0; i < 16; ++i)
                for (int k = 0; k < 32; ++k) {
                    const int q = k / 8, s = k % 8;
                    const int unit = 16 * (2 * kb + s / 4) + 4 * q + s % 4;
                    const int lane = i + 16 * q;
                    tiles[kMlpW2Shorts + ((size_t)(2 * mt + kb) * 64 + lane) * 8 + s] =
                        bf(P[OFF_W2 + unit * kMlpH + 16 * mt + i]);
                }
    for (int ks = 0; ks < 4; ++ks)  // W3^T: rows = outputs (6 used)
        for (int i = 0; i < 16; ++i)
            for (int k = 0; k < 16; ++k)
                put(kMlpW3Tile + ks, i, k, i < kMlpOut ? P[OFF_W3 + (16 * ks + k) * kMlpOut + i] : 0.f);
    bias.assign(kMlpH + kMlpH + 8, 0.f);
    for (int j = 0; j < kMlpH; ++j) {
        bias[j] = P[OFF_B1 + j];
        bias[kMlpH + j] = P[OFF_B2 + j];
    }
    for (int o = 0; o < kMlpOut; ++o) bias[2 * kMlpH + o] = P[OFF_B3 + o];
}

}  // namespace lesasm

using namespace lesasm;

struct lesasm_mlp {
    int device = 0;
    float *params = nullptr, *m = nullptr, *v = nullptr, *grad = nullptr;
    short *packed = nullptr;
    float *bias = nullptr;
    int step = 0;
    // per-workgroup gradient sums of the training kernel, grown on demand
    int cap = 0;  // workgroups
    float *partial = nullptr;
};

static void mlp_free_work(lesasm_mlp *p) {
    device_free(p->partial);
    p->partial = nullptr;
    p->cap = 0;
}

static void mlp_free(lesasm_mlp *p) {
    if (!p) return;
    (void)hipDeviceSynchronize();
    mlp_free_work(p);
    for (void *q : {(void *)p->params, (void *)p->m, (void *)p->v, (void *)p->grad, (void *)p->packed, (void *)p->bias})
        device_free(q);
    delete p;
}

static int mlp_repack(lesasm_mlp *p) {
    std::vector<float> host(kMlpParams);
    LESASM_HIP_TRY(hipMemcpy(host.data(), p->params, sizeof(float) * kMlpParams, hipMemcpyDeviceToHost));
    std::vector<short> tiles;
    std::vector<float> bias;
    pack_weights(host.data(), tiles, bias);
    LESASM_HIP_TRY(hipMemcpy(p->packed, tiles.data(), sizeof(short) * tiles.size(), hipMemcpyHostToDevice));
    LESASM_HIP_TRY(hipMemcpy(p->bias, bias.data(), sizeof(float) * bias.size(), hipMemcpyHostToDevice));
    return LESASM_OK;
}

static int mlp_work(lesasm_mlp *p, int n) {
    const int nb = train_blocks(n);
    if (nb <= p->cap) return LESASM_OK;
    mlp_free_work(p);
    const int st = device_alloc((void **)&p->partial, (size_t)nb * kPartialStride * sizeof(float), "mlp work arrays");
    if (!st) p->cap = nb;
    return st;
}

// Loss and gradients of n samples on s, with room for train_blocks(n) partial sums.
static int launch_train(const lesasm_mlp *p, const float *x, const float *t, int n, float *partial, float *grad,
                        float *loss, hipStream_t s) {
    const int nb = train_blocks(n);
    hipLaunchKernelGGL(k_mlp_train, dim3(nb), dim3(256), sizeof(TrainLds), s, p->params, x, t, n, partial);
    hipLaunchKernelGGL(k_mlp_grad_reduce, dim3((kMlpParams + 1 + 63) / 64), dim3(512), 0, s, partial, nb, grad, loss);
    LESASM_HIP_TRY(hipGetLastError());
    return LESASM_OK;
}

extern "C" int lesasm_mlp_create(const float *params, lesasm_mlp **out) {
    if (!out || !params) return fail(LESASM_E_INVALID_ARG, "mlp_create: NULL argument");
    *out = nullptr;
    auto *p = new lesasm_mlp();
    struct Guard {
        lesasm_mlp *q;
        ~Guard() { mlp_free(q); }
    } guard{p};
    LESASM_HIP_TRY(hipGetDevice(&p->device));
    for (auto pr : {std::make_pair((void **)&p->params, sizeof(float) * kMlpParams),
                    std::make_pair((void **)&p->m, sizeof(float) * kMlpParams),
                    std::make_pair((void **)&p->v, sizeof(float) * kMlpParams),
                    std::make_pair((void **)&p->grad, sizeof(float) * kMlpParams),
                    std::make_pair((void **)&p->packed, sizeof(short) * kMlpPackedShorts),
                    std::make_pair((void **)&p->bias, sizeof(float) * (2 * kMlpH + 8))}) {
        const int st = device_alloc(pr.first, pr.second, "mlp_create");
        if (st) return st;
    }
    LESASM_HIP_TRY(hipMemcpy(p->params, params, sizeof(float) * kMlpParams, hipMemcpyHostToDevice));
    LESASM_HIP_TRY(hipMemset(p->m, 0, sizeof(float) * kMlpParams));
    LESASM_HIP_TRY(hipMemset(p->v, 0, sizeof(float) * kMlpParams));
    int st = mlp_repack(p);
    if (st) return st;
    guard.q = nullptr;
    *out = p;
    return LESASM_OK;
}

extern "C" int lesasm_mlp_destroy(lesasm_mlp *p) {
    mlp_free(p);
    return LESASM_OK;
}

extern "C" int lesasm_mlp_get_params(const lesasm_mlp *p, float *params) {
    if (!p || !params) return fail(LESASM_E_INVALID_ARG, "mlp_get_params: NULL argument");
    LESASM_HIP_TRY(hipMemcpy(params, p->params, sizeof(float) * kMlpParams, hipMemcpyDeviceToHost));
    return LESASM_OK;
}

extern "C" int lesasm_mlp_set_params(lesasm_mlp *p, const float *params) {
    if (!p || !params) return fail(LESASM_E_INVALID_ARG, "mlp_set_params: NULL argument");
    LESASM_HIP_TRY(hipMemcpy(p->params, params, sizeof(float) * kMlpParams, hipMemcpyHostToDevice));
    LESASM_HIP_TRY(hipMemset(p->m, 0, sizeof(float) * kMlpParams));
    LESASM_HIP_TRY(hipMemset(p->v, 0, sizeof(float) * kMlpParams));
    p->step = 0;
    return mlp_repack(p);
}

extern "C" int lesasm_mlp_loss_grad(lesasm_mlp *p, const float *d_x, const float *d_t, int n, float *d_grad,
                                    float *d_loss, void *stream) {
    if (!p || !d_x || !d_t || n < 1) return fail(LESASM_E_INVALID_ARG, "mlp_loss_grad: bad argument");
    int st = mlp_work(p, n);
    if (st) return st;
    return launch_train(p, d_x, d_t, n, p->partial, d_grad ? d_grad : p->grad, d_loss, (hipStream_t)stream);
}

// ---- loss gradient without allocation -------------------------------------------
// The work array of lesasm_mlp_loss_grad_noalloc, the training kernel's partial
// sums for n up to kNoAllocMaxSamples, is one file-scope device array (2.7 MB;
// each device holds its own copy until the process ends).  Host code never
// passes the array's name to a kernel: its device address is taken once per
// device with hipGetSymbolAddress and kept in g_scratch.  Every workgroup
// writes all its sums before any kernel reads them, so nothing is cleared
// between calls.
namespace {
constexpr int kNoAllocMaxSamples = 8192;
constexpr int kNoAllocBlocks = kNoAllocMaxSamples / kTrainTile;
static_assert(kNoAllocMaxSamples % kTrainTile == 0 && kNoAllocBlocks <= kTrainMaxBlocks, "workgroups of the largest call");
constexpr int kScratchDevices = 64;
}  // namespace

static __device__ __align__(256) float scratch[(size_t)kNoAllocBlocks * kPartialStride];

static std::mutex g_scratch_mu;
static float *g_scratch[kScratchDevices];

static int scratch_address(int device, float **out) {
    if (device < 0 || device >= kScratchDevices)
        return fail(LESASM_E_UNSUPPORTED, "mlp_loss_grad_noalloc: device id too large");
    std::lock_guard<std::mutex> lk(g_scratch_mu);
    if (!g_scratch[device]) {
        void *ptr = nullptr;
        const hipError_t e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
        if (e != hipSuccess || !ptr)
            return fail(LESASM_E_HIP, std::string("mlp_loss_grad_noalloc: hipGetSymbolAddress failed: ") +
                                          hipGetErrorString(e));
        g_scratch[device] = (float *)ptr;
    }
    *out = g_scratch[device];
    return LESASM_OK;
}

extern "C" int lesasm_mlp_loss_grad_noalloc(lesasm_mlp *p, const float *d_x, const float *d_t, int n,
                                            float *d_grad, float *d_loss, void *stream) {
    if (!p || !d_x || !d_t || n < 1) return fail(LESASM_E_INVALID_ARG, "mlp_loss_grad_noalloc: bad argument");
    if (n > kNoAllocMaxSamples)
        return fail(LESASM_E_INVALID_ARG, "mlp_loss_grad_noalloc: n = " + std::to_string(n) + " exceeds the " +
                                              std::to_string(kNoAllocMaxSamples) + " samples of the static work area");
    int dev = -1;
    LESASM_HIP_TRY(hipGetDevice(&dev));
    if (dev != p->device) return fail(LESASM_E_STATE, "mlp_loss_grad_noalloc: current device differs from the mlp's");
    float *w = nullptr;
    int st = scratch_address(dev, &w);
    if (st) return st;
    return launch_train(p, d_x, d_t, n, w, d_grad ? d_grad : p->grad, d_loss, (hipStream_t)stream);
}

extern "C" int lesasm_mlp_adam(lesasm_mlp *p, const float *d_grad, float lr, void *stream) {
    if (!p) return fail(LESASM_E_INVALID_ARG, "mlp_adam: NULL argument");
    p->step += 1;
    const float c1 = 1.f - std::pow(0.9f, (float)p->step), c2 = 1.f - std::pow(0.999f, (float)p->step);
    hipLaunchKernelGGL(k_adam, dim3((kMlpParams + 255) / 256), dim3(256), 0, (hipStream_t)stream, p->params, p->m,
                       p->v, d_grad ? d_grad : p->grad, kMlpParams, lr, c1, c2);
    LESASM_HIP_TRY(hipGetLastError());
    return LESASM_OK;
}

extern "C" int lesasm_mlp_train_step(lesasm_mlp *p, const float *d_x, const float *d_t, int n, float lr,
                                     float *d_loss, void *stream) {
    int st = lesasm_mlp_loss_grad(p, d_x, d_t, n, nullptr, d_loss, stream);
    if (st) return st;
    return lesasm_mlp_adam(p, nullptr, lr, stream);
}

extern "C" int lesasm_mlp_commit(lesasm_mlp *p) {
    if (!p) return fail(LESASM_E_INVALID_ARG, "mlp_commit: NULL argument");
    LESASM_HIP_TRY(hipDeviceSynchronize());
    return mlp_repack(p);
}

extern "C" int lesasm_mlp_forward_f32(lesasm_mlp *p, const float *d_x, int n, float *d_y, void *stream) {
    if (!p || !d_x || !d_y || n < 0) return fail(LESASM_E_INVALID_ARG, "mlp_forward_f32: bad argument");
    if (!n) return LESASM_OK;
    // 64 samples a workgroup and round; at most the workgroups that the GPU holds at once (22 KB of LDS each)
    hipLaunchKernelGGL(k_mlp_forward_f32, dim3(std::min((n - 1) / 64 + 1, 1536)), dim3(256), 0, (hipStream_t)stream,
                       p->params, d_x, n, d_y);
    LESASM_HIP_TRY(hipGetLastError());
    return LESASM_OK;
}

extern "C" int lesasm_mlp_infer_bf16(lesasm_mlp *p, const float *d_x, int n, float *d_y, void *stream) {
    if (!p || !d_x || !d_y || n < 0) return fail(LESASM_E_INVALID_ARG, "mlp_infer_bf16: bad argument");
    if (!n) return LESASM_OK;
    const int groups = (n + 63) / 64;
    const int blocks = std::min((groups + 3) / 4, 1024);
    const size_t shm = kMlpLdsBytes + 4 * kMlpWaveScratch;
    hipLaunchKernelGGL(k_mlp_infer_bf16, dim3(blocks), dim3(256), shm, (hipStream_t)stream, p->packed, p->bias, d_x,
                       n, d_y);
    LESASM_HIP_TRY(hipGetLastError());
    return LESASM_OK;
}

// Internal accessors for the fused closure.
namespace lesasm {
const short *mlp_packed(const lesasm_mlp *p) { return p->packed; }
const float *mlp_bias(const lesasm_mlp *p) { return p->bias; }
}  // namespace lesasm
