// Euclidean-time overlaps of a slot's configuration (paper: App. E, the
// tau-dependent Q2, Q4 and F).  For a replica (lane) a and slices tau1,
// tau1 + tau: q_x = S_{x,tau1} S_{x,tau1+tau}, Qt = sum_x q_x, column sums
// C_x1 = sum_x2 q and row sums R_x2 = sum_x1 q.  One launch adds, for every
// requested tau, the integer contributions
//   q2[a][i] += sum_tau1 Qt^2,  q4[a][i] += sum_tau1 Qt^4,
//   A[i][d]  += sum_{a,tau1} sum_x1 C_x1 C_{x1+d},  B[i][d] likewise for R,
// from which Q2, Q4 and F(tau) follow (|sum_x e^{2 pi i x1/L} q_x|^2 =
// sum_d A-term(d) cos(2 pi d/L)).  All sums are integers, so the result does
// not depend on the order of the atomics.
//
// Words hold 64 replicas, so everything up to the products runs on words: a
// lane sums the words of one column (and then of one row) of a slice pair
// into bit-sliced counters u = number of sites with q = -1, C = L - 2u.  The
// lagged products are a contraction over replicas and tau1,
//   U[x][x'] = sum u_x u_x',  sum C_x C_x' = 64 L^2 - 2L (sum u_x + sum u_x') + 4 U,
// and run on the matrix cores: int8 operands, exact 32-bit sums.  A wave
// takes kPlanes slices tau1 at a time, lane (x, i) column x of slice i; a
// matrix operation contracts 16 replicas of each of the wave's slices, and
// since both operands are the same registers the order of replicas within
// them is free: byte b of operand register m holds bit m + 8b of a counter's
// half, which is one shift and one masked or per plane.  The planes'
// transposes across the wave give every replica its total Qt.
//
// What bounds it: vector instructions, about 200 a slice pair and wave at L =
// 16.  A lane per replica, extracting each site's bit and forming the products
// by multiply-adds, took 1800: 142 us for 32 slots, L = 16, L_tau = 128, 14
// tau values, now 30.
#include <hip/hip_runtime.h>

#include <cstdint>

#include "qsg_overlaps.h"

namespace qsg {
namespace {

constexpr int kOvWaves = 4;   // waves per block

typedef int v4i __attribute__((ext_vector_type(4)));
typedef int v16i __attribute__((ext_vector_type(16)));

#define OV_BITOP3(a, b, c, table) __builtin_amdgcn_bitop3_b32((a), (b), (c), (table))

__device__ __forceinline__ uint64_t join(uint32_t lo, uint32_t hi) {
    return (uint64_t)lo | (uint64_t)hi << 32;
}
__device__ __forceinline__ uint64_t xor3(uint64_t a, uint64_t b, uint64_t c) {
    return join(OV_BITOP3((uint32_t)a, (uint32_t)b, (uint32_t)c, 0x96),
                OV_BITOP3((uint32_t)(a >> 32), (uint32_t)(b >> 32), (uint32_t)(c >> 32), 0x96));
}
__device__ __forceinline__ uint64_t majority(uint64_t a, uint64_t b, uint64_t c) {
    return join(OV_BITOP3((uint32_t)a, (uint32_t)b, (uint32_t)c, 0xE8),
                OV_BITOP3((uint32_t)(a >> 32), (uint32_t)(b >> 32), (uint32_t)(c >> 32), 0xE8));
}

constexpr int planes_for(int n) {  // binary digits of n
    int p = 0;
    while (n >> p) ++p;
    return p;
}

// Bit-sliced sum of L words, two at a time: c[0] and the two words by a full
// adder, its carry rippled up.
template <int L, int NP>
__device__ __forceinline__ void count_words(const uint64_t (&w)[L], uint64_t (&c)[NP]) {
#pragma unroll
    for (int p = 0; p < NP; ++p) c[p] = 0;
    static_assert(L % 2 == 0, "words are taken in pairs");
#pragma unroll
    for (int i = 0; i < L; i += 4) {
        // four words: their carries into the twos meet in one adder
        const uint64_t w2 = i + 2 < L ? w[i + 2] : 0, w3 = i + 3 < L ? w[i + 3] : 0;
        const uint64_t ca = majority(c[0], w[i], w[i + 1]);
        c[0] = xor3(c[0], w[i], w[i + 1]);
        const uint64_t cb = majority(c[0], w2, w3);
        c[0] = xor3(c[0], w2, w3);
        uint64_t carry = ca & cb;
        if (NP > 1) {
            carry = majority(c[1], ca, cb);
            c[1] = xor3(c[1], ca, cb);
        }
#pragma unroll
        for (int p = 2; p < NP; ++p) {
            const uint64_t t = c[p] & carry;
            c[p] ^= carry;
            carry = t;
        }
    }
}

// Operand register m of a counter half: byte b = the counter of bit m + 8b.
template <int NP>
__device__ __forceinline__ uint32_t counter_bytes(const uint32_t (&c)[NP], int m) {
    uint32_t r = (c[0] >> m) & 0x01010101u;
#pragma unroll
    for (int p = 1; p < NP; ++p) {
        const uint32_t v = m >= p ? c[p] >> (m - p) : c[p] << (p - m);
        r = OV_BITOP3(v, 0x01010101u << p, r, 0xEA);  // (v & mask) | r
    }
    return r;
}

// The matrix accumulator of U: X x X, symmetric, lane l column l % X.
template <int X> struct Products;
template <> struct Products<16> {
    static constexpr int kRows = 4;
    v4i d = {};
    __device__ __forceinline__ void add(v4i a) {
        d = __builtin_amdgcn_mfma_i32_16x16x64_i8(a, a, d, 0, 0, 0);
    }
    __device__ __forceinline__ static int row(int r, int lane) { return 4 * (lane >> 4) + r; }
};
template <> struct Products<32> {
    static constexpr int kRows = 16;
    v16i d = {};
    __device__ __forceinline__ void add(v4i a) {
        d = __builtin_amdgcn_mfma_i32_32x32x32_i8(a, a, d, 0, 0, 0);
    }
    __device__ __forceinline__ static int row(int r, int lane) {
        return 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3);
    }
};

template <int NP, int X>
__device__ __forceinline__ void add_products(const uint64_t (&c)[NP], Products<X>& u) {
    uint32_t half[2][NP];
#pragma unroll
    for (int p = 0; p < NP; ++p) {
        half[0][p] = (uint32_t)c[p];
        half[1][p] = (uint32_t)(c[p] >> 32);
    }
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int m = 0; m < 8; m += 4) {
            v4i a;
#pragma unroll
            for (int k = 0; k < 4; ++k) a[k] = (int)counter_bytes(half[h], m + k);
            u.add(a);
        }
}

// 64 x 64 bit transpose across the wave: afterwards thread t holds, in bit
// b, bit t of thread b's word (stage k swaps bit k of the thread index with
// bit k of the bit index).
__device__ __forceinline__ uint64_t transpose(uint64_t x, uint32_t t) {
    uint32_t lo = (uint32_t)x, hi = (uint32_t)(x >> 32);
    {
        const bool up = (t & 32u) != 0;
        const uint32_t recv = (uint32_t)__shfl_xor((int)(up ? lo : hi), 32, 64);
        lo = up ? recv : lo;
        hi = up ? hi : recv;
    }
    constexpr uint32_t kHigh[5] = {0xAAAAAAAAu, 0xCCCCCCCCu, 0xF0F0F0F0u, 0xFF00FF00u, 0xFFFF0000u};
#pragma unroll
    for (int k = 4; k >= 0; --k) {
        const uint32_t sh = 1u << k;
        const bool up = (t & sh) != 0;
        const uint32_t keep = up ? kHigh[k] : ~kHigh[k];
        const uint32_t rot = up ? sh : 32u - sh;
        const uint32_t ylo = (uint32_t)__shfl_xor((int)lo, (int)sh, 64);
        const uint32_t yhi = (uint32_t)__shfl_xor((int)hi, (int)sh, 64);
        lo = OV_BITOP3(keep, lo, __builtin_amdgcn_alignbit(ylo, ylo, rot), 0xCA);
        hi = OV_BITOP3(keep, hi, __builtin_amdgcn_alignbit(yhi, yhi, rot), 0xCA);
    }
    return join(lo, hi);
}

// Order the wave's own LDS accesses before and after.
__device__ __forceinline__ void wave_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// kGroups: groups of kPlanes slices per wave.
template <int L, int kGroups>
__global__ void __launch_bounds__(64 * kOvWaves)
k_tau_overlaps(const uint64_t* __restrict__ spins, uint32_t Ltau, TauList taus,
               int64_t* __restrict__ out) {
    constexpr int P = L * L;
    constexpr int X = L <= 16 ? 16 : 32;   // lanes per slice
    constexpr int kPlanes = 64 / X;        // slices per wave
    constexpr int NP = planes_for(L);
    constexpr uint32_t kPerBlock = kOvWaves * kGroups * kPlanes;
    // q of the wave's slices (rows padded: a lane then reads its row without
    // bank conflicts); at the end the accumulators
    constexpr int kQ = kPlanes * L * (L + 1), kU = (2 * X * X + 1) / 2;
    __shared__ uint64_t lds[kOvWaves][kQ > kU ? kQ : kU];
    __shared__ int64_t red2[kOvWaves][64], red4[kOvWaves][64];
    __shared__ int64_t redn[kOvWaves];
    // blockIdx.z: the slot, counted from the first one requested; each slot
    // has its own output block q2 [64][n], q4 [64][n], A [n][L], B [n][L]
    const uint64_t* __restrict__ S = spins + (size_t)blockIdx.z * P * Ltau;
    int64_t* __restrict__ q2o = out + (size_t)blockIdx.z * taus.n * (128 + 2 * L);
    int64_t* __restrict__ q4o = q2o + 64 * (size_t)taus.n;
    int64_t* __restrict__ Ao = q4o + 64 * (size_t)taus.n;
    int64_t* __restrict__ Bo = Ao + (size_t)taus.n * L;
    const uint32_t lane = threadIdx.x & 63u;
    const uint32_t w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const uint32_t x = lane % X, plane = lane / X;
    const uint32_t it = blockIdx.y;
    const uint32_t tau = taus.t[it];
    Products<X> ua, ub;
    int64_t s2 = 0, s4 = 0;
    int32_t ones = 0, slices = 0;  // sites with q = -1 of this replica; slices counted
#pragma unroll 1
    for (uint32_t k = 0; k < kGroups; ++k) {
        const uint32_t first = blockIdx.x * kPerBlock + (k * kOvWaves + w) * kPlanes;
        if (first >= Ltau) break;
        const uint32_t tau1 = first + plane;
        const bool have = x < (uint32_t)L && tau1 < Ltau;
        uint64_t v[L], c[NP];
        if (have) {
            uint32_t tau2 = tau1 + tau;
            if (tau2 >= Ltau) tau2 -= Ltau;
            const uint64_t* __restrict__ a = S + (size_t)tau1 * P + x;
            const uint64_t* __restrict__ b = S + (size_t)tau2 * P + x;
#pragma unroll
            for (int y = 0; y < L; ++y) v[y] = a[y * L] ^ b[y * L];
            uint64_t* q = &lds[w][plane * L * (L + 1) + x];
#pragma unroll
            for (int y = 0; y < L; ++y) q[y * (L + 1)] = v[y];
        } else {
#pragma unroll
            for (int y = 0; y < L; ++y) v[y] = 0;
        }
        count_words<L, NP>(v, c);  // the column
        add_products(c, ua);
        // totals per replica and slice: bit x + X i of the transposed planes
        int32_t total[kPlanes] = {};
#pragma unroll
        for (int p = 0; p < NP; ++p) {
            const uint64_t z = transpose(c[p], lane);
#pragma unroll
            for (int i = 0; i < kPlanes; ++i)
                total[i] += __popc((uint32_t)(z >> (X * i)) & (X == 32 ? ~0u : 0xFFFFu)) << p;
        }
#pragma unroll
        for (int i = 0; i < kPlanes; ++i) {
            if (first + i >= Ltau) break;
            const int64_t qt = P - 2 * total[i];
            const int64_t sq = qt * qt;
            s2 += sq;
            s4 += sq * sq;
            ones += total[i];
            ++slices;
        }
        // the row of the same index, through LDS (the wave's own region:
        // no other wave is waited for)
        wave_sync();
        if (have) {
            const uint64_t* q = &lds[w][(plane * L + x) * (L + 1)];
#pragma unroll
            for (int i = 0; i < L; ++i) v[i] = q[i];
        }
        wave_sync();
        count_words<L, NP>(v, c);
        add_products(c, ub);
    }
    // the block's accumulators and totals; lds now holds U of columns, rows
    int32_t* u = reinterpret_cast<int32_t*>(&lds[w][0]);
#pragma unroll
    for (int r = 0; r < Products<X>::kRows; ++r) {
        const int at = Products<X>::row(r, (int)lane) * X + (int)x;
        u[at] = ua.d[r];
        u[X * X + at] = ub.d[r];
    }
    red2[w][lane] = s2;
    red4[w][lane] = s4;
    int64_t n1 = ones;
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) n1 += __shfl_xor(n1, off, 64);
    // sum over x of (64 L^2 - 4 L u_x) over the wave's slices
    if (lane == 0) redn[w] = (int64_t)slices * 64 * L * P - 4 * L * n1;
    __syncthreads();
    if (w == 0) {
        int64_t t2 = 0, t4 = 0;
#pragma unroll
        for (int k = 0; k < kOvWaves; ++k) {
            t2 += red2[k][lane];
            t4 += red4[k][lane];
        }
        atomicAdd((unsigned long long*)&q2o[(size_t)lane * taus.n + it], (unsigned long long)t2);
        atomicAdd((unsigned long long*)&q4o[(size_t)lane * taus.n + it], (unsigned long long)t4);
    } else if (w < 3 && lane < (uint32_t)L) {  // wave 1: columns, wave 2: rows; lag = lane
        int64_t sum = 0;
#pragma unroll
        for (int k = 0; k < kOvWaves; ++k) {
            const int32_t* m = reinterpret_cast<const int32_t*>(&lds[k][0]) + (w - 1) * X * X;
            int64_t part = 0;
            for (int i = 0; i < L; ++i) part += m[i * X + (i + (int)lane) % L];
            sum += redn[k] + 4 * part;
        }
        atomicAdd((unsigned long long*)&(w == 1 ? Ao : Bo)[(size_t)it * L + lane],
                  (unsigned long long)sum);
    }
}

template <int L, int kGroups>
hipError_t launch_groups(const uint64_t* slot_spins, uint32_t n_slots, uint32_t Ltau,
                         const TauList& taus, int64_t* out, hipStream_t s) {
    constexpr uint32_t kPerBlock = kOvWaves * kGroups * (L <= 16 ? 4 : 2);
    const dim3 grid((Ltau + kPerBlock - 1) / kPerBlock, taus.n, n_slots);
    hipLaunchKernelGGL((k_tau_overlaps<L, kGroups>), grid, dim3(64 * kOvWaves), 0, s, slot_spins, Ltau,
                       taus, out);
    return hipGetLastError();
}

// A wave takes two groups of slices before its block adds to the output, and
// four where the planes are so small that adding is most of the work and the
// blocks of two groups fill the chip several times (L = 2: 142 -> 85 us on 16384
// blocks, 10.2 -> 9.0 on 896, but 4.5 -> 7.2 on 64; L = 4: 120 -> 92 on 16384,
// 20.3 -> 17.3 on 2048; a lane per replica took 131, 9.5, 4.6, 107 and 19.5).
template <int L>
hipError_t launch_width(const uint64_t* slot_spins, uint32_t n_slots, uint32_t Ltau,
                        const TauList& taus, int64_t* out, hipStream_t s) {
    if constexpr (L <= 4) {
        const uint64_t blocks = (uint64_t)((Ltau + 31) / 32) * taus.n * n_slots;
        if (blocks >= (L == 2 ? 512 : 2048))
            return launch_groups<L, 4>(slot_spins, n_slots, Ltau, taus, out, s);
    }
    return launch_groups<L, 2>(slot_spins, n_slots, Ltau, taus, out, s);
}

}  // namespace

hipError_t launch_tau_overlaps(const uint64_t* slot_spins, uint32_t n_slots, uint32_t L,
                               uint32_t Ltau, const TauList& taus, int64_t* out, hipStream_t s) {
    if (taus.n == 0 || n_slots == 0) return hipSuccess;
    switch (L) {
#define QSG_OV_WIDTH(W) \
    case W: return launch_width<W>(slot_spins, n_slots, Ltau, taus, out, s);
        QSG_OV_WIDTH(2) QSG_OV_WIDTH(4) QSG_OV_WIDTH(6) QSG_OV_WIDTH(8) QSG_OV_WIDTH(10)
        QSG_OV_WIDTH(12) QSG_OV_WIDTH(14) QSG_OV_WIDTH(16) QSG_OV_WIDTH(18) QSG_OV_WIDTH(20)
        QSG_OV_WIDTH(22) QSG_OV_WIDTH(24) QSG_OV_WIDTH(26) QSG_OV_WIDTH(28) QSG_OV_WIDTH(30)
        QSG_OV_WIDTH(32)
#undef QSG_OV_WIDTH
        default: return hipErrorInvalidValue;
    }
}

}  // namespace qsg
