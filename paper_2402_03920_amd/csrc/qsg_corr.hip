// Correlations of transfer-matrix eigenvectors (paper: App. E, the
// consistency checks of EDQSG): Q2, Q4 and F of a slice need the
// Walsh-Hadamard transform of v^2 only at the sets of one to four bits (pairs
// and quadruples of the L^2 sites; a set that holds the last site has a bit
// less): 12 950 of 2^24 entries at L = 5.  So the transform is pruned:
//
//   k_corr_low: the low 12 index bits of each 4096-state tile, of which only
//     the 794 entries of at most four bits are kept (a fifth of the tile); at
//     L = 5 a block takes eight tiles and does the three bits that number
//     them as well, so that it writes whole 64-byte sectors;
//   k_corr_high: for each kept low entry the other bits, then the sums over
//     its sets of R R' (see qsg_corr.h), one partial row per block;
//   k_corr_sum: the rows in order.
//
// L <= 3 (at most 256 states) takes one block, k_corr_small.
//
// The vector is read once and 26 MB of it written and read again: at L = 5
// what bounds the call is that read (134 MB; two vectors for the estimates at
// finite lengths), of which 72 us of k_corr_low reach 3.7 TB/s: its three LDS
// exchanges a tile (occupancies of four blocks a CU, or four tiles a block,
// measured 74 to 85 us).  The whole transform by the product's two passes,
// each reading and writing the vector, a one-block gather of the entries and
// their table built on the host made an estimate from two vectors 416 us; now
// 163, of them 106 in these kernels.
#include <hip/hip_runtime.h>

#include <cmath>
#include <cstdint>

#include "qsg_corr.h"
#include "qsg_transfer.h"

namespace qsg {
namespace {

constexpr int kThreads = 256;
constexpr int kTile = 4096;       // entries a block transforms at once
constexpr int kPad = kTile / 16;  // LDS padding: element e at e + e / 16
constexpr int kMaxBits = 4;

constexpr int bits_of(int v) { return v == 0 ? 0 : (v & 1) + bits_of(v >> 1); }
constexpr int count_low() {
    int n = 0;
    for (int v = 0; v < kTile; ++v) n += bits_of(v) <= kMaxBits;
    return n;
}
constexpr int kLow = count_low();  // 1 + 12 + 66 + 220 + 495

// The 12-bit values of at most four bits, ascending.
struct LowTable {
    uint16_t value[kLow];
};
constexpr LowTable make_low() {
    LowTable t{};
    int n = 0;
    for (int v = 0; v < kTile; ++v)
        if (bits_of(v) <= kMaxBits) t.value[n++] = (uint16_t)v;
    return t;
}
__constant__ LowTable c_low = make_low();
static_assert(kLow == 794, "sets of at most four of twelve bits");

template <int R>
__device__ __forceinline__ void hadamard(double (&x)[R], int first = 1) {
#pragma unroll
    for (int q = 1; q < R; q <<= 1) {
        if (q < first) continue;
#pragma unroll
        for (int r = 0; r < R; ++r) {
            if (r & q) continue;
            const double a = x[r], b = x[r | q];
            x[r] = a + b;
            x[r | q] = a - b;
        }
    }
}

// Walsh-Hadamard transform of 4096 values by 256 threads: thread t holds
// values 16 t + r on entry (register bits already done by the caller) and
// values t + 256 q on return.
__device__ __forceinline__ void transform_tile(double* lds, double (&x)[16]) {
    const uint32_t t = threadIdx.x;
    const uint32_t lo = t & 15, hi = t >> 4;
#pragma unroll
    for (int r = 0; r < 16; ++r) lds[17 * t + r] = x[r];
    __syncthreads();
#pragma unroll
    for (int s = 0; s < 16; ++s) x[s] = lds[lo + 17 * (s + 16 * hi)];
    hadamard(x);
#pragma unroll
    for (int s = 0; s < 16; ++s) lds[lo + 17 * (s + 16 * hi)] = x[s];
    __syncthreads();
#pragma unroll
    for (int q = 0; q < 16; ++q) x[q] = lds[t + 256 * q + ((t + 256 * q) >> 4)];
    hadamard(x);
}

// Sum over the block, in every thread.
__device__ __forceinline__ double block_total(double v, double* red) {
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
    __syncthreads();
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
    __syncthreads();
    double s = 0.0;
#pragma unroll
    for (int i = 0; i < kThreads / 64; ++i) s += red[i];
    return s;
}

// Low bits.  Block x takes tiles x T ... x T + T - 1 of the vector of
// blockIdx.y; out: per vector [kLow][M], M = tiles of the vector.  With T =
// 8 the transform over the tile's low three bits is done too.
template <int T>
__global__ void __launch_bounds__(kThreads)
k_corr_low(const double* __restrict__ even, const double* __restrict__ odd, uint32_t M,
           double* __restrict__ out) {
    __shared__ double lds[kTile + kPad];
    constexpr int kPer = (kLow + kThreads - 1) / kThreads;  // kept entries per thread
    const uint32_t t = threadIdx.x;
    const double* __restrict__ v = blockIdx.y ? odd : even;
    double* __restrict__ dst = out + (size_t)blockIdx.y * kLow * M;
    const uint32_t first = blockIdx.x * T;
    uint32_t pos[kPer];
#pragma unroll
    for (int i = 0; i < kPer; ++i) {
        const uint32_t j = t + kThreads * i;
        const uint32_t e = c_low.value[j < kLow ? j : 0];
        pos[i] = e + (e >> 4);
    }
    auto load = [&](uint32_t tile, double (&x)[16]) {
        const size_t base = (size_t)tile * kTile + 16 * t;
#pragma unroll
        for (int r = 0; r < 16; r += 2) {
            const double2 a = *reinterpret_cast<const double2*>(v + base + r);
            x[r] = a.x;
            x[r + 1] = a.y;
        }
    };
    double keep[kPer][T], next[16];
    load(first, next);
#pragma unroll
    for (int k = 0; k < T; ++k) {
        double x[16];
#pragma unroll
        for (int r = 0; r < 16; ++r) x[r] = next[r] * next[r];
        if (k + 1 < T) load(first + k + 1, next);  // in flight during this tile
        hadamard(x);
        transform_tile(lds, x);
        __syncthreads();
#pragma unroll
        for (int q = 0; q < 16; ++q) lds[t + 256 * q + ((t + 256 * q) >> 4)] = x[q];
        __syncthreads();
#pragma unroll
        for (int i = 0; i < kPer; ++i) keep[i][k] = lds[pos[i]];
        __syncthreads();
    }
#pragma unroll
    for (int i = 0; i < kPer; ++i) {
        const uint32_t j = t + kThreads * i;
        if (j >= kLow) continue;
        hadamard(keep[i]);
#pragma unroll
        for (int k = 0; k < T; ++k) dst[(size_t)j * M + first + k] = keep[i][k];
    }
}

struct CosTable {
    double c[kTmMaxL];  // cos(2 pi d / L)
};

// Adds a set's products R R' to the sums (the set as its bits, the last site
// left out; nothing for other than one to four bits).
template <bool kMixed>
__device__ __forceinline__ void add_set(uint32_t set, uint32_t L, double re, double ro,
                                        const double* cosl, double (&sum)[kCorrSums]) {
    const uint32_t c = (uint32_t)__popc(set);
    if (c == 0 || c > kMaxBits) return;
    const double rr[3] = {re * re, re * ro, ro * ro};
    if (c > 2) {
#pragma unroll
        for (int k = 0; k < (kMixed ? 3 : 1); ++k) sum[3 * k + 2] += rr[k];
        return;
    }
    const uint32_t a = 31u - (uint32_t)__clz(set);
    const uint32_t b = c == 1 ? L * L - 1 : (uint32_t)__ffs(set) - 1;
    const int d1 = (int)(a % L) - (int)(b % L), d2 = (int)(a / L) - (int)(b / L);
    const double w = cosl[abs(d1)] + cosl[abs(d2)];
#pragma unroll
    for (int k = 0; k < (kMixed ? 3 : 1); ++k) {
        sum[3 * k] += rr[k];
        sum[3 * k + 1] += w * rr[k];
    }
}

// At most 256 states: one block, a state per thread, a round per index bit
// through LDS.
template <bool kMixed>
__global__ void __launch_bounds__(kThreads)
k_corr_small(const double* __restrict__ even, const double* __restrict__ odd, uint32_t L,
             CosTable cosines, double* __restrict__ out) {
    __shared__ double v[2][kThreads], red[kThreads / 64], cosl[kTmMaxL];
    const uint32_t t = threadIdx.x, n = L * L - 1, N = 1u << n;
    if (t < kTmMaxL) cosl[t] = cosines.c[t];
    double e = t < N ? even[t] : 0.0, o = kMixed && t < N ? odd[t] : 0.0;
    e *= e;
    o *= o;
    for (uint32_t j = 0; j < n; ++j) {
        __syncthreads();
        v[0][t] = e;
        if (kMixed) v[1][t] = o;
        __syncthreads();
        const uint32_t s = t ^ (1u << j);
        const bool up = (t >> j) & 1u;
        e = up ? v[0][s] - e : e + v[0][s];
        if (kMixed) o = up ? v[1][s] - o : o + v[1][s];
    }
    __syncthreads();
    if (t == 0) {
        v[0][0] = e;
        v[1][0] = o;
    }
    __syncthreads();
    double sum[kCorrSums] = {};
    if (t < N) add_set<kMixed>(t, L, e * (1.0 / v[0][0]), kMixed ? o * (1.0 / v[1][0]) : 0.0, cosl, sum);
#pragma unroll
    for (int k = 0; k < (kMixed ? kCorrSums : 3); ++k) {
        const double s = block_total(sum[k], red);
        if (t == 0) out[k] = s;
    }
}

// High bits and sums: block j the kept low entry j.
template <int T, bool kMixed>
__global__ void __launch_bounds__(kThreads)
k_corr_high(const double* __restrict__ C, uint32_t L, uint32_t M, CosTable cosines,
            double* __restrict__ partial) {
    __shared__ double lds[kTile + kPad];
    __shared__ double red[kThreads / 64];
    __shared__ double cosl[kTmMaxL];
    const uint32_t t = threadIdx.x;
    if (t < kTmMaxL) cosl[t] = cosines.c[t];
    const size_t vec = (size_t)kLow * M;
    // W[0] of a vector: the low entry 0 over all tiles (one of every T, the
    // others are differences within a group)
    auto norm = [&](const double* c) {
        double s = 0.0;
        for (uint32_t h = t * T; h < M; h += kThreads * T) s += c[h];
        return 1.0 / block_total(s, red);
    };
    const double inv_e = norm(C), inv_o = kMixed ? norm(C + vec) : 0.0;
    double sum[kCorrSums] = {};
    const uint32_t j = blockIdx.x, low = c_low.value[j];
    auto load = [&](const double* c, double (&x)[16]) {
        const double* p = c + (size_t)j * M + 16 * t;
        if (M == kTile) {
#pragma unroll
            for (int r = 0; r < 16; r += 2) {
                const double2 a = *reinterpret_cast<const double2*>(p + r);
                x[r] = a.x;
                x[r + 1] = a.y;
            }
        } else {  // fewer tiles: the rest is zero
#pragma unroll
            for (int r = 0; r < 16; ++r) x[r] = 16 * t + r < M ? p[r] : 0.0;
        }
    };
    double e[16], o[16];
    load(C, e);
    if (kMixed) load(C + vec, o);
    hadamard(e, T);
    transform_tile(lds, e);
    if (kMixed) {
        __syncthreads();  // lds is used again
        hadamard(o, T);
        transform_tile(lds, o);
    }
#pragma unroll
    for (int q = 0; q < 16; ++q) {
        const uint32_t h = t + 256 * q;
        if (h < M)
            add_set<kMixed>(h << 12 | low, L, e[q] * inv_e, kMixed ? o[q] * inv_o : 0.0, cosl, sum);
    }
#pragma unroll
    for (int k = 0; k < (kMixed ? kCorrSums : 3); ++k) {
        const double s = block_total(sum[k], red);
        if (t == 0) partial[(size_t)blockIdx.x * kCorrSums + k] = s;
    }
}

// out[k] = sum of the rows' entries k.
__global__ void __launch_bounds__(kThreads)
k_corr_sum(const double* __restrict__ partial, uint32_t rows, uint32_t n, double* __restrict__ out) {
    __shared__ double red[kThreads / 64];
    double v = 0.0;
    for (uint32_t i = threadIdx.x; i < rows; i += kThreads) v += partial[(size_t)i * kCorrSums + blockIdx.x];
    const double s = block_total(v, red);
    if (threadIdx.x == 0) out[blockIdx.x] = s;
}

uint32_t tiles_of(uint32_t L) { return (1u << (L * L - 1)) / kTile; }  // 0: one block does it

template <int T>
void launch_corr(uint32_t M, uint32_t L, const double* even, const double* odd, double* ws,
                 double* partial, const CosTable& cosines, hipStream_t s) {
    hipLaunchKernelGGL(k_corr_low<T>, dim3(M / T, odd ? 2 : 1), dim3(kThreads), 0, s, even, odd, M, ws);
    if (odd)
        hipLaunchKernelGGL((k_corr_high<T, true>), dim3(kLow), dim3(kThreads), 0, s, ws, L, M, cosines,
                           partial);
    else
        hipLaunchKernelGGL((k_corr_high<T, false>), dim3(kLow), dim3(kThreads), 0, s, ws, L, M,
                           cosines, partial);
}

}  // namespace

size_t tm_corr_ws_doubles(uint32_t L, bool mixed) {
    const size_t M = tiles_of(L);
    return M ? (mixed ? 2 : 1) * kLow * M + (size_t)kLow * kCorrSums : 0;
}

hipError_t launch_tm_corr_sums(uint32_t L, const double* even, const double* odd, double* ws,
                               double* out, hipStream_t s) {
    const uint32_t M = tiles_of(L);
    CosTable cosines;
    for (uint32_t d = 0; d < kTmMaxL; ++d)
        cosines.c[d] = std::cos(6.283185307179586476925286766559 * d / L);
    if (M == 0) {
        if (odd)
            hipLaunchKernelGGL(k_corr_small<true>, dim3(1), dim3(kThreads), 0, s, even, odd, L, cosines,
                               out);
        else
            hipLaunchKernelGGL(k_corr_small<false>, dim3(1), dim3(kThreads), 0, s, even, odd, L,
                               cosines, out);
        return hipGetLastError();
    }
    double* partial = ws + (size_t)(odd ? 2 : 1) * kLow * M;
    // eight tiles a block where that leaves two blocks a CU (L = 5)
    if (M >= 4096) launch_corr<8>(M, L, even, odd, ws, partial, cosines, s);
    else launch_corr<1>(M, L, even, odd, ws, partial, cosines, s);
    const uint32_t sums = odd ? kCorrSums : 3;
    hipLaunchKernelGGL(k_corr_sum, dim3(sums), dim3(kThreads), 0, s, partial, (uint32_t)kLow, sums, out);
    return hipGetLastError();
}

}  // namespace qsg
