// Ladder-predicting MLP: forward, backward, loss, Adam and ladder decode.
//
// Network 6 -> 128 -> 128 -> 128 -> 32 with exact-erf GELU after the hidden
// layers.  Parameters are FP32 master values (flat layout W1[6][128], b1,
// W2[128][128], b2, W3[128][128], b3, W4[128][32], b4; W[k][n] maps input k
// to output n) with an optional BF16 copy.  With the BF16 copy, every GEMM
// operand is rounded to bfloat16 (nearest even) and products accumulate in
// FP32; bias, GELU, loss and Adam are FP32.  Without it the same kernels run
// in FP32 throughout.
//
// The matrices are at most [B x 128] x [128 x 128]: what costs time is the
// latency of launches and of the weight reads, not arithmetic.  So a pass is
// one launch whose blocks keep all weights in registers, read up front, and
// take a few samples at a time through all layers.  The sums of the forward
// pass and of the data gradients run over the inputs in order, because with
// BF16 operands a last-bit difference in one layer is rounded to another
// operand in the next.  Everything is deterministic (no float atomics).
#include <hip/hip_runtime.h>

#include <cmath>
#include <cstdint>
#include <mutex>

#include "qsg_mlp.h"

namespace qsg {
namespace {

__device__ __forceinline__ float bf16_round(float x) {
    uint32_t u = __float_as_uint(x);
    u += 0x7FFFu + ((u >> 16) & 1u);
    return __uint_as_float(u & 0xFFFF0000u);
}
__device__ __forceinline__ float bf16_to_f32(uint16_t h) {
    return __uint_as_float((uint32_t)h << 16);
}
__device__ __forceinline__ uint16_t f32_to_bf16(float x) {
    return (uint16_t)(__float_as_uint(bf16_round(x)) >> 16);
}
__device__ __forceinline__ float gelu(float x) {
    return 0.5f * x * (1.0f + erff(x * 0.70710678118654752f));
}
__device__ __forceinline__ float gelu_grad(float x) {
    return 0.5f * (1.0f + erff(x * 0.70710678118654752f)) +
           x * expf(-0.5f * x * x) * 0.39894228040143268f;
}

struct Layer {
    int K, N;
    size_t w_off, b_off;
};

__host__ __device__ inline Layer layer(int l) {
    const int K[4] = {kMlpIn, kMlpHidden, kMlpHidden, kMlpHidden};
    const int N[4] = {kMlpHidden, kMlpHidden, kMlpHidden, kMlpOut};
    size_t off = 0;
    for (int i = 0; i < l; ++i) off += (size_t)K[i] * N[i] + N[i];
    return Layer{K[l], N[l], off, off + (size_t)K[l] * N[l]};
}

// Operand of a product: rounded to bfloat16 when the BF16 copy is in use.
template <bool kHalf>
__device__ __forceinline__ float operand(float x) {
    return kHalf ? bf16_round(x) : x;
}

// Weight number i of the FP32 master or of the BF16 copy.
template <bool kHalf>
__device__ __forceinline__ float weight(const float* __restrict__ pf,
                                        const uint16_t* __restrict__ ph, size_t i) {
    return kHalf ? bf16_to_f32(ph[i]) : pf[i];
}

// A block is three groups of 128 threads; each thread keeps the 128 weights
// of one output of one layer in registers, so that all weight reads of the
// network are in flight together and are read once per block (one launch per
// layer, each reading its weights in its own dependent loop, took 12 us a
// layer; the whole pass now takes 8.5 us up to 512 samples and 11 at 1024,
// before 42 to 47).  Blocks then loop over tiles of S samples: one as long as every
// sample can have a block of its own on a CU (256 of them), then 2, 4 and 8,
// which share the barriers between layers.
constexpr int kGroup = kMlpHidden;
constexpr int kGroups = 3;
constexpr int kMlpBlocks = 256;
constexpr int kMaxTile = 8;

inline int tile_samples(int B) {
    int s = 1;
    while (s < kMaxTile && B > s * kMlpBlocks) s *= 2;
    return s;
}

// a0 = sum_k v0[k] w[k], a1 = sum_k v1[k] w[k] (v0, v1 in LDS), in order of k.
__device__ __forceinline__ void dot2(const float* v0, const float* v1,
                                     const float (&w)[kMlpHidden], float& a0, float& a1) {
    a0 = a1 = 0.0f;
#pragma unroll
    for (int k = 0; k < kMlpHidden; k += 4) {
        const float4 x = *reinterpret_cast<const float4*>(v0 + k);
        const float4 y = *reinterpret_cast<const float4*>(v1 + k);
        a0 = fmaf(x.x, w[k], a0);
        a1 = fmaf(y.x, w[k], a1);
        a0 = fmaf(x.y, w[k + 1], a0);
        a1 = fmaf(y.y, w[k + 1], a1);
        a0 = fmaf(x.z, w[k + 2], a0);
        a1 = fmaf(y.z, w[k + 2], a1);
        a0 = fmaf(x.w, w[k + 3], a0);
        a1 = fmaf(y.w, w[k + 3], a1);
        // not all of v ahead in registers: the weights need them
        if (k % 32 == 28) asm volatile("" : "+v"(a0), "+v"(a1) : : "memory");
    }
}

// Forward pass, S samples a tile.  Group 0 does layer 1, group 1 layer 2,
// group 2 layers 0 and 3 (output n & 31 of every fourth sample).
template <bool kHalf>
__global__ void __launch_bounds__(kGroups * kGroup)
k_forward(const float* __restrict__ X, int B, int S, const float* __restrict__ pf,
          const uint16_t* __restrict__ ph, float* __restrict__ ws, float* __restrict__ out) {
    __shared__ __align__(16) float h[3][kMaxTile][kMlpHidden];  // operands of layers 1, 2, 3
    __shared__ float xin[kMaxTile][kMlpIn];
    const int group = __builtin_amdgcn_readfirstlane((int)threadIdx.x / kGroup);
    const int n = (int)threadIdx.x % kGroup;
    const Layer L = layer(group + 1);
    const int col = group == 2 ? n % kMlpOut : n;
    float w[kMlpHidden], w0[kMlpIn];
#pragma unroll
    for (int k = 0; k < kMlpIn; ++k) w0[k] = weight<kHalf>(pf, ph, layer(0).w_off + k * kMlpHidden + n);
#pragma unroll
    for (int k = 0; k < kMlpHidden; ++k)
        w[k] = weight<kHalf>(pf, ph, L.w_off + (size_t)k * L.N + col);
    const float bias = pf[L.b_off + col], bias0 = pf[layer(0).b_off + n];
    const int tiles = (B + S - 1) / S;
    for (int tile = blockIdx.x; tile < tiles; tile += gridDim.x) {
        const int b0 = tile * S, left = min(S, B - b0);
        if ((int)threadIdx.x < left * kMlpIn)
            xin[threadIdx.x / kMlpIn][threadIdx.x % kMlpIn] =
                operand<kHalf>(X[(size_t)b0 * kMlpIn + threadIdx.x]);
        __syncthreads();
        auto put = [&](int l, int s, float pre) {  // a hidden layer's result of sample s
            const float act = gelu(pre);
            h[l][s][n] = operand<kHalf>(act);
            ws[mlp_ws_pre(l, B) + (size_t)(b0 + s) * kMlpHidden + n] = pre;
            ws[mlp_ws_act(l, B) + (size_t)(b0 + s) * kMlpHidden + n] = act;
        };
        if (group == 2) {
#pragma unroll 1
            for (int s = 0; s < left; ++s) {
                float acc = 0.0f;
#pragma unroll
                for (int k = 0; k < kMlpIn; ++k) acc = fmaf(xin[s][k], w0[k], acc);
                put(0, s, acc + bias0);
            }
        }
        __syncthreads();
#pragma unroll 1
        for (int l = 1; l < 3; ++l) {
            if (group == l - 1) {
#pragma unroll 1
                for (int s = 0; s < left; s += 2) {
                    const int s1 = min(s + 1, left - 1);
                    float a0, a1;
                    dot2(h[l - 1][s], h[l - 1][s1], w, a0, a1);
                    put(l, s, a0 + bias);
                    if (s1 > s) put(l, s1, a1 + bias);
                }
            }
            __syncthreads();
        }
        if (group == 2) {
            const int s0 = n / kMlpOut, s1 = s0 + kMlpHidden / kMlpOut;
            float a0, a1;
            if (s0 < left) {
                dot2(h[2][s0], h[2][s1 < left ? s1 : s0], w, a0, a1);
                out[(size_t)(b0 + s0) * kMlpOut + col] = a0 + bias;
                if (s1 < left) out[(size_t)(b0 + s1) * kMlpOut + col] = a1 + bias;
            }
        }
        // the next tile's first writes are to xin and h[0], which no thread
        // reads past the last barrier
    }
}

// Gradients of the pre-activations of the hidden layers: gpre_l[k] =
// (sum_n g_{l+1}[n] W_{l+1}[k][n]) gelu'(pre_l[k]), from the output's
// gradient down.  Group 0 does layer 2, group 1 layer 1, group 2 layer 0,
// each thread with its row of the weights in registers.  Layer 2's stay in
// the block (the weight gradients form them again: the caller's scratch
// holds two of the three).
template <bool kHalf>
__global__ void __launch_bounds__(kGroups * kGroup)
k_backward_data(const float* __restrict__ dout, int B, int S, const float* __restrict__ pf,
                const uint16_t* __restrict__ ph, const float* __restrict__ ws,
                float* __restrict__ gpre1, float* __restrict__ gpre0) {
    __shared__ __align__(16) float g3[kMaxTile][kMlpOut];
    __shared__ __align__(16) float g[2][kMaxTile][kMlpHidden];  // operands of layers 2 and 1
    __shared__ float slope[kGroups][kMaxTile][kMlpHidden];      // gelu'(pre) of the group's layer
    const int group = __builtin_amdgcn_readfirstlane((int)threadIdx.x / kGroup);
    const int k = (int)threadIdx.x % kGroup;
    const int l = 2 - group;
    const Layer L = layer(l + 1);
    float w[kMlpHidden];  // group 0: its row has 32
    if (group == 0) {
#pragma unroll
        for (int n = 0; n < kMlpOut; ++n) w[n] = weight<kHalf>(pf, ph, L.w_off + (size_t)k * kMlpOut + n);
    } else {
#pragma unroll
        for (int n = 0; n < kMlpHidden; ++n)
            w[n] = weight<kHalf>(pf, ph, L.w_off + (size_t)k * kMlpHidden + n);
    }
    float* gout = group == 1 ? gpre1 : gpre0;
    const int tiles = (B + S - 1) / S;
    for (int tile = blockIdx.x; tile < tiles; tile += gridDim.x) {
        const int b0 = tile * S, left = min(S, B - b0);
        if ((int)threadIdx.x < left * kMlpOut)
            g3[threadIdx.x / kMlpOut][threadIdx.x % kMlpOut] =
                operand<kHalf>(dout[(size_t)b0 * kMlpOut + threadIdx.x]);
#pragma unroll 1
        for (int s = 0; s < left; ++s)
            slope[group][s][k] = gelu_grad(ws[mlp_ws_pre(l, B) + (size_t)(b0 + s) * kMlpHidden + k]);
        __syncthreads();
        if (group == 0) {
#pragma unroll 1
            for (int s = 0; s < left; ++s) {
                float acc = 0.0f;
#pragma unroll
                for (int n = 0; n < kMlpOut; ++n) acc = fmaf(g3[s][n], w[n], acc);
                g[0][s][k] = operand<kHalf>(acc * slope[0][s][k]);
            }
        }
        __syncthreads();
#pragma unroll 1
        for (int step = 0; step < 2; ++step) {
            if (group == step + 1) {
                auto put = [&](int s, float sum) {
                    const float v = sum * slope[group][s][k];
                    if (step == 0) g[1][s][k] = operand<kHalf>(v);
                    gout[(size_t)(b0 + s) * kMlpHidden + k] = v;
                };
#pragma unroll 1
                for (int s = 0; s < left; s += 2) {
                    const int s1 = min(s + 1, left - 1);
                    float a0, a1;
                    dot2(g[step][s], g[step][s1], w, a0, a1);
                    put(s, a0);
                    if (s1 > s) put(s1, a1);
                }
            }
            __syncthreads();
        }
    }
}

// Weight and bias gradients of all layers in one launch: dW[k][n] = sum_b
// x[b][k] g[b][n], db[n] = sum_b g[b][n].  A block of 16 waves forms a 32 x
// 32 tile of one layer's dW over all samples, 128 samples at a time staged in
// LDS: each wave takes 8 of them, each lane a 4 x 4 piece of the tile, and
// the waves' sums are added in order at the end.  What costs time is the
// latency of a round of reads, so a round is large and a thread has its reads
// in flight together: 16 us at 321 samples, 26 with rounds of 32.  (A thread
// per output that walked the batch alone, layer by layer with the data
// gradients between, made a training step of 321 samples 490 us; now 42.)
constexpr int kDwTile = 32;
constexpr int kDwWaves = 16;
constexpr int kDwThreads = 64 * kDwWaves;
constexpr int kDwRows = 4;                                       // staged per thread
constexpr int kDwChunk = kDwRows * kDwThreads / kDwTile;         // samples per round
constexpr int kDwPerWave = kDwChunk / kDwWaves;
// blocks of layer l: (K / 32 rounded up) x (N / 32)
constexpr int dw_blocks(int l) {
    return l == 0 ? kMlpHidden / kDwTile
         : l < 3  ? (kMlpHidden / kDwTile) * (kMlpHidden / kDwTile)
                  : (kMlpHidden / kDwTile) * (kMlpOut / kDwTile);
}
constexpr int kDwBlocks = dw_blocks(0) + dw_blocks(1) + dw_blocks(2) + dw_blocks(3);

template <bool kHalf>
__global__ void __launch_bounds__(kDwThreads)
k_backward_weight(const float* __restrict__ X, const float* __restrict__ dout, int B,
                  const float* __restrict__ pf, const uint16_t* __restrict__ ph,
                  const float* __restrict__ ws, const float* __restrict__ gpre1,
                  const float* __restrict__ gpre0, float* __restrict__ grads) {
    // the staged samples, then the waves' sums
    __shared__ __align__(16) float lds[kDwWaves * kDwTile * kDwTile];
    static_assert(3 * kDwChunk <= kDwWaves * kDwTile, "the operands fit");
    float(*xs)[kDwTile] = reinterpret_cast<float(*)[kDwTile]>(lds);
    float(*gs)[kDwTile] = xs + kDwChunk;
    float(*ds)[kDwTile] = gs + kDwChunk;  // layer 2: the output's gradients
    __shared__ float bpart[kDwTile][kDwTile];
    int block = blockIdx.x, l = 0;
    while (block >= dw_blocks(l)) block -= dw_blocks(l++);
    const Layer L = layer(l);
    const int ntiles = L.N / kDwTile;
    const int k0 = block / ntiles * kDwTile, n0 = block % ntiles * kDwTile;
    const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
    const int row = t >> 5, c = t & 31;  // staging: sample `row` of the 32, column c
    const float* x = l == 0 ? X : ws + mlp_ws_act(l - 1, B);
    const float* g = l == 3 ? dout : l == 1 ? gpre1 : gpre0;
    float w3[kMlpOut];  // layer 2: this column's row of the output weights
    if (l == 2) {
#pragma unroll
        for (int n = 0; n < kMlpOut; ++n)
            w3[n] = weight<kHalf>(pf, ph, layer(3).w_off + (size_t)(n0 + c) * kMlpOut + n);
    }
    const int ky = lane >> 3, nx = lane & 7;
    float acc[4][4] = {};
    float db = 0.0f;
    for (int b0 = 0; b0 < B; b0 += kDwChunk) {
        float xv[kDwRows], gv[kDwRows];
#pragma unroll
        for (int i = 0; i < kDwRows; ++i) {
            const int b = b0 + row + kDwTile * i;
            xv[i] = gv[i] = 0.0f;
            if (b >= B) continue;
            if (k0 + c < L.K) xv[i] = x[(size_t)b * L.K + k0 + c];
            if (l == 2)
                gv[i] = ws[mlp_ws_pre(2, B) + (size_t)b * kMlpHidden + n0 + c];
            else
                gv[i] = g[(size_t)b * L.N + n0 + c];
        }
        if (l == 2) {  // gv holds gelu's argument: form the gradient from the output's
            static_assert(kMlpOut == kDwTile, "one output column per staging column");
#pragma unroll
            for (int i = 0; i < kDwRows; ++i) {
                const int b = b0 + row + kDwTile * i;
                ds[row + kDwTile * i][c] =
                    b < B ? operand<kHalf>(dout[(size_t)b * kMlpOut + c]) : 0.0f;
            }
            __syncthreads();
#pragma unroll
            for (int i = 0; i < kDwRows; ++i) {
                float s = 0.0f;
#pragma unroll
                for (int n = 0; n < kMlpOut; n += 4) {
                    const float4 v = *reinterpret_cast<const float4*>(&ds[row + kDwTile * i][n]);
                    s = fmaf(v.x, w3[n], s);
                    s = fmaf(v.y, w3[n + 1], s);
                    s = fmaf(v.z, w3[n + 2], s);
                    s = fmaf(v.w, w3[n + 3], s);
                }
                // nothing where the batch has ended (0 times an infinite weight is not 0)
                gv[i] = b0 + row + kDwTile * i < B ? s * gelu_grad(gv[i]) : 0.0f;
                asm volatile("" : "+v"(gv[i]) : : "memory");  // one row's reads at a time
            }
        }
        __syncthreads();  // the previous round's samples are used up
#pragma unroll
        for (int i = 0; i < kDwRows; ++i) {
            xs[row + kDwTile * i][c] = operand<kHalf>(xv[i]);
            gs[row + kDwTile * i][c] = operand<kHalf>(gv[i]);
            db += gv[i];
        }
        __syncthreads();
#pragma unroll
        for (int i = 0; i < kDwPerWave; ++i) {
            const float4 a = *reinterpret_cast<const float4*>(&xs[kDwPerWave * wave + i][4 * ky]);
            const float4 d = *reinterpret_cast<const float4*>(&gs[kDwPerWave * wave + i][4 * nx]);
            const float av[4] = {a.x, a.y, a.z, a.w}, dv[4] = {d.x, d.y, d.z, d.w};
#pragma unroll
            for (int p = 0; p < 4; ++p)
#pragma unroll
                for (int q = 0; q < 4; ++q) acc[p][q] = fmaf(av[p], dv[q], acc[p][q]);
        }
    }
    __syncthreads();  // the staging buffers become the waves' sums
#pragma unroll
    for (int p = 0; p < 4; ++p)
        *reinterpret_cast<float4*>(&lds[(wave * kDwTile + 4 * ky + p) * kDwTile + 4 * nx]) =
            make_float4(acc[p][0], acc[p][1], acc[p][2], acc[p][3]);
    bpart[row][c] = db;
    __syncthreads();
    float sum = 0.0f;
#pragma unroll
    for (int v = 0; v < kDwWaves; ++v) sum += lds[v * kDwTile * kDwTile + t];
    if (k0 + row < L.K) grads[L.w_off + (size_t)(k0 + row) * L.N + n0 + c] = sum;
    if (k0 == 0 && t < kDwTile) {
        float s = 0.0f;
#pragma unroll
        for (int v = 0; v < kDwTile; ++v) s += bpart[v][t];
        grads[L.b_off + n0 + t] = s;
    }
}

// Loss and decode take 32 threads per sample (a half wave): thread l its
// logit's exponentials and logarithms; the sums run over the logits in order
// in every thread, from LDS.  That is short where it leaves the chip idle, but
// repeats every sum 32 times: larger batches take a thread per sample, with
// the same operations in the same order.  32 threads / one (us): loss 4.0 /
// 5.2 on one sample, 4.9 / 6.1 on 4096, 5.6 / 6.2 on 8192, 8.8 / 6.4 on 16384,
// 24 / 12 on 65536; decode 9.1 on 8192, 15 / 11 on 16384, 51 / 15 on 65536.
constexpr int kRowSamples = 8;  // samples per block of 256 threads
constexpr int kRowBatch = 8192;

__device__ __forceinline__ float row_max(float v) {
#pragma unroll
    for (int off = 16; off > 0; off >>= 1) v = fmaxf(v, __shfl_xor(v, off, 32));
    return v;
}

// Per sample: KL(t || softmax(z[:31])) + (z[31] - logL)^2 and its gradient,
// scaled by 1/B (mean over the batch).
__global__ void __launch_bounds__(32 * kRowSamples)
k_loss(const float* __restrict__ z, const float* __restrict__ t, const float* __restrict__ logL,
       int B, float* __restrict__ dz, float* __restrict__ loss) {
    __shared__ float es[kRowSamples][kMlpOut], ts[kRowSamples][kMlpOut], as[kRowSamples][kMlpOut];
    const int r = threadIdx.x >> 5, l = threadIdx.x & 31;
    const int b = blockIdx.x * kRowSamples + r;
    const bool head = l == kMlpInc;  // the barrier head
    float zl = 0.0f, tl = 0.0f;
    if (b < B) {
        zl = z[(size_t)b * kMlpOut + l];
        if (!head) tl = t[(size_t)b * kMlpInc + l];
    }
    const float m = row_max(head ? -INFINITY : zl);
    es[r][l] = expf(zl - m);
    ts[r][l] = tl;
    __syncthreads();
    float se = 0.0f, tsum = 0.0f;
#pragma unroll
    for (int i = 0; i < kMlpInc; ++i) {
        se += es[r][i];
        tsum += ts[r][i];
    }
    const float lse = m + logf(se);
    const float inv_b = 1.0f / (float)B;
    const float d = head && b < B ? zl - logL[b] : 0.0f;
    if (b < B)
        dz[(size_t)b * kMlpOut + l] =
            head ? 2.0f * d * inv_b : (expf(zl - lse) * tsum - tl) * inv_b;
    as[r][l] = tl > 0.0f ? logf(tl) - (zl - lse) : 0.0f;
    __syncthreads();
    if (head && b < B) {
        float kl = 0.0f;
#pragma unroll
        for (int i = 0; i < kMlpInc; ++i)
            if (ts[r][i] > 0.0f) kl = fmaf(ts[r][i], as[r][i], kl);
        loss[b] = kl + d * d;
    }
}

__global__ void __launch_bounds__(64)
k_loss_by_sample(const float* __restrict__ z, const float* __restrict__ t,
                 const float* __restrict__ logL, int B, float* __restrict__ dz,
                 float* __restrict__ loss) {
    const int b = blockIdx.x * 64 + threadIdx.x;
    if (b >= B) return;
    const float* zb = z + (size_t)b * kMlpOut;
    const float* tb = t + (size_t)b * kMlpInc;
    float m = -INFINITY;
    for (int l = 0; l < kMlpInc; ++l) m = fmaxf(m, zb[l]);
    float se = 0.0f, tsum = 0.0f;
    for (int l = 0; l < kMlpInc; ++l) {
        se += expf(zb[l] - m);
        tsum += tb[l];
    }
    const float lse = m + logf(se);
    const float inv_b = 1.0f / (float)B;
    const float d = zb[kMlpInc] - logL[b];
    float kl = 0.0f;
    for (int l = 0; l < kMlpInc; ++l) {
        const float zl = zb[l], tl = tb[l];
        if (tl > 0.0f) kl = fmaf(tl, logf(tl) - (zl - lse), kl);
        dz[(size_t)b * kMlpOut + l] = (expf(zl - lse) * tsum - tl) * inv_b;
    }
    dz[(size_t)b * kMlpOut + kMlpInc] = 2.0f * d * inv_b;
    loss[b] = kl + d * d;
}

__global__ void k_adam(float* __restrict__ p, uint16_t* __restrict__ ph, const float* __restrict__ g,
                       float* __restrict__ m, float* __restrict__ v, int n, float lr, float c1,
                       float c2) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const float gi = g[i];
    const float mi = 0.9f * m[i] + 0.1f * gi;
    const float vi = 0.999f * v[i] + 0.001f * gi * gi;
    m[i] = mi;
    v[i] = vi;
    const float pi = p[i] - lr * (mi / c1) / (sqrtf(vi / c2) + 1e-8f);
    p[i] = pi;
    if (ph) ph[i] = f32_to_bf16(pi);
}

__global__ void k_to_bf16(const float* __restrict__ p, uint16_t* __restrict__ ph, int n) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) ph[i] = f32_to_bf16(p[i]);
}

// Ladder from the 31 increment logits: log G_i = log Gmin + (log Gmax -
// log Gmin) * cumulative softmax, non-decreasing, ends pinned exactly;
// predicted acceptance 1 - exp(z31)/31.  Thread l forms point l + 1.  (Ends
// given the wrong way round, Gmin > Gmax, keep Gmin up to the last inner
// point, which like the end is Gmax.)
__global__ void __launch_bounds__(32 * kRowSamples)
k_decode(const float* __restrict__ z, const double* __restrict__ gmin,
         const double* __restrict__ gmax, int B, double* __restrict__ ladder,
         float* __restrict__ acc_pred) {
    __shared__ double es[kRowSamples][kMlpOut];
    const int r = threadIdx.x >> 5, l = threadIdx.x & 31;
    const int b = blockIdx.x * kRowSamples + r;
    const bool head = l == kMlpInc;
    const float zl = b < B ? z[(size_t)b * kMlpOut + l] : 0.0f;
    const double m = row_max(head ? -INFINITY : zl);
    es[r][l] = exp((double)zl - m);
    __syncthreads();
    double se = 0.0;
#pragma unroll
    for (int i = 0; i < kMlpInc; ++i) se += es[r][i];
    double c = 0.0;
#pragma unroll
    for (int i = 0; i < kMlpInc; ++i)
        if (i <= l) c += es[r][i] / se;
    const double first = b < B ? gmin[b] : 1.0, last = b < B ? gmax[b] : 1.0;
    const double lo = log(first), hi = log(last);
    double v = exp(lo + (hi - lo) * c);  // (comparisons that leave a NaN in place)
    if (v < first) v = first;
    if (last >= first && v > last) v = last;
#pragma unroll
    for (int off = 1; off < 32; off <<= 1) {  // running maximum over the points
        const double below = __shfl_up(v, off, 32);
        if (l >= off && below > v) v = below;
    }
    if (l == kMlpInc - 2 && v > last) v = last;
    if (b >= B) return;
    double* out = ladder + (size_t)b * kMlpLadder;
    if (head) {
        out[0] = first;
        if (acc_pred) acc_pred[b] = 1.0f - expf(zl) / (float)kMlpInc;
    } else {
        out[l + 1] = l == kMlpInc - 1 ? last : v;
    }
}

__global__ void __launch_bounds__(64)
k_decode_by_sample(const float* __restrict__ z, const double* __restrict__ gmin,
                   const double* __restrict__ gmax, int B, double* __restrict__ ladder,
                   float* __restrict__ acc_pred) {
    const int b = blockIdx.x * 64 + threadIdx.x;
    if (b >= B) return;
    const float* zb = z + (size_t)b * kMlpOut;
    float m = -INFINITY;
    for (int l = 0; l < kMlpInc; ++l) m = fmaxf(m, zb[l]);
    double se = 0.0;
    for (int l = 0; l < kMlpInc; ++l) se += exp((double)zb[l] - (double)m);
    const double first = gmin[b], last = gmax[b];
    const double lo = log(first), hi = log(last);
    double* out = ladder + (size_t)b * kMlpLadder;
    const double cap = last >= first ? last : INFINITY;
    double c = 0.0, v = first;
    out[0] = first;
#pragma unroll 6
    for (int l = 0; l < kMlpInc - 1; ++l) {  // the exponentials of six points side by side
        c += exp((double)zb[l] - (double)m) / se;
        double next = exp(lo + (hi - lo) * c);
        if (next > cap) next = cap;
        if (v > next) next = v;
        out[l + 1] = v = next;
    }
    if (v > last) out[kMlpLadder - 2] = last;
    out[kMlpLadder - 1] = last;
    if (acc_pred) acc_pred[b] = 1.0f - expf(zb[kMlpInc]) / (float)kMlpInc;
}

inline unsigned blocks(long n, int t) { return (unsigned)((n + t - 1) / t); }

}  // namespace

namespace {

template <bool kHalf>
void launch_forward(const float* pf, const uint16_t* ph, const float* x, int B, float* out,
                    float* ws, hipStream_t s) {
    const int S = tile_samples(B);
    hipLaunchKernelGGL(k_forward<kHalf>, dim3(min((B + S - 1) / S, kMlpBlocks)),
                       dim3(kGroups * kGroup), 0, s, x, B, S, pf, ph, ws, out);
}

template <bool kHalf>
void launch_backward(const float* pf, const uint16_t* ph, const float* x, const float* ws,
                     const float* dout, int B, float* grads, float* gpre1, float* gpre0,
                     hipStream_t s) {
    const int S = tile_samples(B);
    hipLaunchKernelGGL(k_backward_data<kHalf>, dim3(min((B + S - 1) / S, kMlpBlocks)),
                       dim3(kGroups * kGroup), 0, s, dout, B, S, pf, ph, ws, gpre1, gpre0);
    hipLaunchKernelGGL(k_backward_weight<kHalf>, dim3(kDwBlocks), dim3(kDwThreads), 0, s, x, dout, B,
                       pf, ph, ws, gpre1, gpre0, grads);
}

}  // namespace

hipError_t mlp_forward(const float* pf, const uint16_t* ph, const float* x, int B, float* out,
                       float* ws, hipStream_t s) {
    if (ph) launch_forward<true>(pf, ph, x, B, out, ws, s);
    else launch_forward<false>(pf, ph, x, B, out, ws, s);
    return hipGetLastError();
}

hipError_t mlp_backward(const float* pf, const uint16_t* ph, const float* x, const float* ws,
                        const float* dout, int B, float* grads, float* scratch, hipStream_t s) {
    // scratch: [B][128] twice, the pre-activation gradients of layers 1 and 0
    float* gpre1 = scratch;
    float* gpre0 = scratch + (size_t)B * kMlpHidden;
    if (ph) launch_backward<true>(pf, ph, x, ws, dout, B, grads, gpre1, gpre0, s);
    else launch_backward<false>(pf, ph, x, ws, dout, B, grads, gpre1, gpre0, s);
    return hipGetLastError();
}

hipError_t mlp_loss(const float* z, const float* t, const float* logL, int B, float* dz,
                    float* loss, hipStream_t s) {
    if (B <= kRowBatch)
        hipLaunchKernelGGL(k_loss, dim3(blocks(B, kRowSamples)), dim3(32 * kRowSamples), 0, s, z, t,
                           logL, B, dz, loss);
    else
        hipLaunchKernelGGL(k_loss_by_sample, dim3(blocks(B, 64)), dim3(64), 0, s, z, t, logL, B, dz,
                           loss);
    return hipGetLastError();
}

hipError_t mlp_adam(float* p, uint16_t* ph, const float* g, float* m, float* v, uint32_t step,
                    float lr, hipStream_t s) {
    const float c1 = 1.0f - powf(0.9f, (float)step);
    const float c2 = 1.0f - powf(0.999f, (float)step);
    hipLaunchKernelGGL(k_adam, dim3(blocks(kMlpParams, 256)), dim3(256), 0, s, p, ph, g, m, v,
                       kMlpParams, lr, c1, c2);
    return hipGetLastError();
}

hipError_t mlp_to_bf16(const float* p, uint16_t* ph, hipStream_t s) {
    hipLaunchKernelGGL(k_to_bf16, dim3(blocks(kMlpParams, 256)), dim3(256), 0, s, p, ph, kMlpParams);
    return hipGetLastError();
}

hipError_t mlp_decode(const float* z, const double* gmin, const double* gmax, int B, double* ladder,
                      float* acc_pred, hipStream_t s) {
    if (B <= kRowBatch)
        hipLaunchKernelGGL(k_decode, dim3(blocks(B, kRowSamples)), dim3(32 * kRowSamples), 0, s, z,
                           gmin, gmax, B, ladder, acc_pred);
    else
        hipLaunchKernelGGL(k_decode_by_sample, dim3(blocks(B, 64)), dim3(64), 0, s, z, gmin, gmax, B,
                           ladder, acc_pred);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Forward pass that allocates nothing: the activations live in a fixed
// device array of this library (one copy per GPU, held until the process
// ends) instead of a caller workspace.  In host code `scratch` names a
// host-side stand-in, not the device copy: its device address comes from
// hipGetSymbolAddress, looked up once per device with that device current,
// and only that address is ever passed to kernels.
// ---------------------------------------------------------------------------
__device__ __align__(256) float scratch[(size_t)kMlpNoAllocMaxBatch * (6 * kMlpHidden + kMlpOut)];
static_assert(sizeof(scratch) / sizeof(float) >= (size_t)6 * kMlpNoAllocMaxBatch * kMlpHidden +
                                                       (size_t)kMlpNoAllocMaxBatch * kMlpOut,
              "scratch must hold the forward workspace of the largest batch");

namespace {
constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
float* g_scratch_ptr[kMaxDevices] = {};
}  // namespace

hipError_t mlp_noalloc_scratch(float** out) {
    int dev = -1;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lock(g_scratch_mu);
    if (!g_scratch_ptr[dev]) {
        void* p = nullptr;
        e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess) return e;
        g_scratch_ptr[dev] = static_cast<float*>(p);
    }
    *out = g_scratch_ptr[dev];
    return hipSuccess;
}

hipError_t mlp_forward_noalloc(const float* pf, const uint16_t* ph, const float* x, int B,
                               float* out, hipStream_t s) {
    float* ws = nullptr;
    hipError_t e = mlp_noalloc_scratch(&ws);
    if (e != hipSuccess) return e;
    return mlp_forward(pf, ph, x, B, out, ws, s);
}

}  // namespace qsg
