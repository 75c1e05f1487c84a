// HIP kernels (gfx950, wave64) of the MCQSG Metropolis + parallel-tempering
// hot path.  Paper: Sec. 2.1 (multi-spin coding, checkerboard Metropolis,
// precomputed acceptance factors, parallel tempering), Sec. 2.1.1 (counter-
// based Philox4x32-10 random numbers tied to the lattice update).
//
// Multi-spin coding here packs 64 independent chains of one site into a
// uint64 (bit j = lane j), so a thread updates 64 spins with bitwise logic:
//   * unsatisfied bonds: u = s ^ neighbour ^ J (bit set <=> J S S' < 0);
//   * per-lane counts n_s (4 space bonds) and n_t (2 time bonds) as
//     bit-sliced adders, turned into a three-bit class code;
//   * acceptance r_j <= thr[class_j]: lane numbers are bit-sliced over 32
//     levels (bit 31-b of r_j is bit j of level b), so all 64 comparisons run
//     together, most significant level first, and stop as soon as every lane
//     of the wave is decided.  One Philox block yields two levels.
// The sweeps hold no contraction, so there is no matrix-core work here: they
// are integer VALU work on data streamed from HBM (or held in LDS).
#include <hip/hip_runtime.h>

#include "qsg_internal.h"

namespace qsg {
namespace {

constexpr uint32_t kM0 = 0xD2511F53u;
constexpr uint32_t kM1 = 0xCD9E8D57u;
constexpr uint32_t kW0 = 0x9E3779B9u;
constexpr uint32_t kW1 = 0xBB67AE85u;

// Philox4x32-10 (Salmon et al., SC'11): ten rounds of two 32x32->64 products
// and xors with the key, the key advanced by the Weyl constants.  Each
// product is one v_mad_u64_u32 (both halves at once) and each three-way xor
// one v_bitop3_b32.
__device__ __forceinline__ uint32_t xor3(uint32_t a, uint32_t b, uint32_t c) {
    return __builtin_amdgcn_bitop3_b32(a, b, c, 0x96);
}

// Where only counter word 0 differs between lanes, the first two rounds group
// their xors to keep the uniform parts on the scalar unit: round 0 has c.y,
// c.z, c.w uniform, round 1 c.x, c.y.
__device__ __forceinline__ uint4 philox(uint4 c, uint32_t k0, uint32_t k1) {
#pragma unroll
    for (int r = 0; r < 10; ++r) {
        const uint64_t p0 = (uint64_t)c.x * kM0;
        const uint64_t p1 = (uint64_t)c.z * kM1;
        const uint32_t h0 = (uint32_t)(p0 >> 32), h1 = (uint32_t)(p1 >> 32);
        if (r == 0)
            c = make_uint4(h1 ^ (c.y ^ k0), (uint32_t)p1, h0 ^ (c.w ^ k1), (uint32_t)p0);
        else if (r == 1)
            c = make_uint4(h1 ^ (c.y ^ k0), (uint32_t)p1, (h0 ^ k1) ^ c.w, (uint32_t)p0);
        else
            c = make_uint4(xor3(h1, c.y, k0), (uint32_t)p1, xor3(h0, c.w, k1), (uint32_t)p0);
        k0 += kW0;
        k1 += kW1;
    }
    return c;
}

// The same block in two parts for the colour pass, where counter word 0 (the
// site) differs between lanes and words 1-3 (sweep, slot and block, group)
// are block-uniform.  What only the site, the group and the key decide is
// kept per word over its blocks (philox_site: round 0's product of the site
// and round 1's product of its high half); per block (philox_block) the
// uniform products of the first two rounds run on the scalar unit, which
// leaves 2 + 8 * 4 vector instructions.
struct PhiloxSite {
    uint32_t lo0;       // low half of round 0's product of the site
    uint32_t lo1, hi1;  // round 1's product of (its high half ^ group ^ key)
};

__device__ __forceinline__ PhiloxSite philox_site(uint32_t s, uint32_t gid, uint32_t k1) {
    const uint64_t p = (uint64_t)s * kM0;
    const uint64_t q = (uint64_t)((uint32_t)(p >> 32) ^ (gid ^ k1)) * kM1;
    return {(uint32_t)p, (uint32_t)q, (uint32_t)(q >> 32)};
}

__device__ __forceinline__ uint4 philox_block(const PhiloxSite& ps, uint32_t t, uint32_t gq,
                                              uint32_t k0, uint32_t k1) {
    const uint64_t u = (uint64_t)gq * kM1;                                // round 0
    const uint64_t v = (uint64_t)((uint32_t)(u >> 32) ^ t ^ k0) * kM0;    // round 1
    uint4 c = make_uint4(ps.hi1 ^ ((uint32_t)u ^ (k0 + kW0)), ps.lo1,
                         ps.lo0 ^ ((uint32_t)(v >> 32) ^ (k1 + kW1)), (uint32_t)v);
#pragma unroll
    for (int r = 2; r < 10; ++r) {
        k0 += r == 2 ? 2 * kW0 : kW0;
        k1 += r == 2 ? 2 * kW1 : kW1;
        const uint64_t p0 = (uint64_t)c.x * kM0;
        const uint64_t p1 = (uint64_t)c.z * kM1;
        const uint32_t h0 = (uint32_t)(p0 >> 32), h1 = (uint32_t)(p1 >> 32);
        if (r == 2)  // c.w is uniform
            c = make_uint4(xor3(h1, c.y, k0), (uint32_t)p1, h0 ^ (c.w ^ k1), (uint32_t)p0);
        else
            c = make_uint4(xor3(h1, c.y, k0), (uint32_t)p1, xor3(h0, c.w, k1), (uint32_t)p0);
    }
    return c;
}

__device__ __forceinline__ uint64_t lo_hi(uint32_t lo, uint32_t hi) {
    return (uint64_t)lo | ((uint64_t)hi << 32);
}

// A group record read from memory by a batched kernel: every block reads one
// record, so its fields are block-uniform; moving them to scalar registers
// keeps all addressing and threshold logic on the scalar unit.
__device__ __forceinline__ GroupDev uniform_record(const GroupDev* __restrict__ p) {
    static_assert(sizeof(GroupDev) % 4 == 0, "record must be whole dwords");
    union {
        GroupDev g;
        uint32_t w[sizeof(GroupDev) / 4];
    } u;
    u.g = *p;
#pragma unroll
    for (int i = 0; i < (int)(sizeof(GroupDev) / 4); ++i) u.w[i] = __builtin_amdgcn_readfirstlane(u.w[i]);
    return u.g;
}

// Division of x < 2^31 by a block-uniform d >= 1 with a precomputed
// multiplier: q = mulhi(x, m) >> s (see make_divisor on the host).
__device__ __forceinline__ uint32_t fast_div(uint32_t x, Divisor d) {
    return d.m ? (__umulhi(x, d.m) >> d.s) : (x >> d.s);
}

// Three-input bitwise operation of gfx950 (v_bitop3_b32); the immediate is
// the truth table f(0xF0, 0xCC, 0xAA) of the operand order (a, b, c).
#define BITOP3(a, b, c, table) __builtin_amdgcn_bitop3_b32((a), (b), (c), (table))
constexpr int kAndXnor = 0x90;    // a & ~(b ^ c)
constexpr int kXor3 = 0x96;       // a ^ b ^ c
constexpr int kMajority = 0xE8;   // at least two of a, b, c
constexpr int kXorAnd = 0x78;     // a ^ (b & c)
constexpr int kXorAndNot = 0xB4;  // a ^ (b & ~c)
constexpr int kSelect = 0xCA;     // a ? b : c (bitwise)
constexpr int kAnd3 = 0x80;       // a & b & c
constexpr int kNotEq3 = 0x7E;     // not (a == b and a == c)
constexpr int kNeNe = 0x18;       // a != b and a != c

template <int T>
__device__ __forceinline__ uint64_t bop3(uint64_t a, uint64_t b, uint64_t c) {
    return lo_hi(BITOP3((uint32_t)a, (uint32_t)b, (uint32_t)c, T),
                 BITOP3((uint32_t)(a >> 32), (uint32_t)(b >> 32), (uint32_t)(c >> 32), T));
}

// A word under update: site, centre word, the class code of every lane as
// three bit planes (code = p2 p1 p0, see class_code) and the lanes the
// comparison still has to decide (at first those whose flip can raise the
// energy).
struct Word {
    uint32_t s;  // flat site index (RNG counter word 0)
    uint64_t w;  // centre word, accepted lanes already flipped
    uint64_t p0, p1, p2;
    uint64_t und;
};

// LDS of a colour-pass block: the words still undecided after the first
// levels, packed by all threads of the block and finished by as few waves as
// possible.  Two pairs of counters alternate between consecutive calls of a
// block: a slow thread may still be reading the previous call's count after
// a fast one has cleared the counters for the next call.
struct SweepQueue {
    uint32_t count[4];
    uint32_t s[kSweepBlock];
    uint64_t w[kSweepBlock], p0[kSweepBlock], p1[kSweepBlock], p2[kSweepBlock];
    uint64_t und[kSweepBlock];
};

// The four couplings of every thread's column (column walk).
struct WalkCouplings {
    uint64_t xp[kSweepBlock], xm[kSweepBlock], yp[kSweepBlock], ym[kSweepBlock];
};

// Spin and coupling words are addressed as base + 32-bit byte offset, so
// global accesses keep the base in SGPRs and only the offset in a VGPR.  The
// host rejects slots of more than 2^29 words, so a word index i < 2^29 gives
// a byte offset i * 8 < 2^32.  The fused kernel may hold a slot in LDS.
typedef char __attribute__((address_space(1))) GlobalByte;
template <bool kGlobal>
__device__ __forceinline__ uint64_t load64(const uint64_t* base, uint32_t i) {
    if (kGlobal)
        return *(const uint64_t __attribute__((address_space(1)))*)((const GlobalByte*)base + i * 8u);
    return base[i];
}
template <bool kGlobal>
__device__ __forceinline__ void store64(uint64_t* base, uint32_t i, uint64_t v) {
    if (kGlobal)
        *(uint64_t __attribute__((address_space(1)))*)((GlobalByte*)base + i * 8u) = v;
    else
        base[i] = v;
}

// Unsatisfied space bonds u = w ^ neighbour ^ coupling of a word, counted per
// lane: n_s = s2 s1 s0, a full adder over u1..u3, then u4 added to its sum.
struct SpaceCount {
    uint64_t s0, s1, s2;
};
__device__ __forceinline__ SpaceCount count_space(uint64_t w, uint64_t nxp, uint64_t nxm,
                                                  uint64_t nyp, uint64_t nym, uint64_t jxp,
                                                  uint64_t jxm, uint64_t jyp, uint64_t jym) {
    const uint64_t u1 = bop3<kXor3>(w, nxp, jxp), u2 = bop3<kXor3>(w, nxm, jxm);
    const uint64_t u3 = bop3<kXor3>(w, nyp, jyp), u4 = bop3<kXor3>(w, nym, jym);
    const uint64_t sum = bop3<kXor3>(u1, u2, u3), carry = bop3<kMajority>(u1, u2, u3);
    return {sum ^ u4, bop3<kXorAnd>(carry, sum, u4), bop3<kAnd3>(carry, sum, u4)};
}

// Class codes.  A flip can raise the energy (dE > 0) in at most seven of the
// fifteen classes (n_s, n_t), and which seven depends only on the ordering of
// the two couplings (the regime; every other class is accepted outright):
//   regime 0 (kp > 2k):        n_t = 0: n_s = 0..4;  n_t = 1: n_s = 0, 1
//   regime 1 (k < kp <= 2k):   n_t = 0: n_s = 0..3;  n_t = 1: n_s = 0, 1;  n_t = 2: n_s = 0
//   regime 2 (kp <= k):        n_t = 0: n_s = 0..2;  n_t = 1, 2: n_s = 0, 1
// Three planes number the seven classes 0..6 (kClassCode of the host lists
// the same codes), so that any function of the class, such as the threshold
// bits of one level, is one three-input operation on them.  und: the lanes
// in one of the seven classes; the codes of the others are not used.
__device__ __forceinline__ Word class_code(uint32_t regime, uint32_t s, uint64_t w,
                                           const SpaceCount& n, uint64_t above, uint64_t below) {
    Word r;
    r.s = s;
    r.w = w;
    const uint64_t nt1 = above ^ below;
    const uint64_t some = bop3<kNotEq3>(w, above, below);  // n_t > 0
    if (regime == 0) {  // n_t = 0: n_s; n_t = 1: 5 + n_s
        asm volatile("");  // a block-uniform branch, not a select of both sides
        r.p0 = n.s0 ^ nt1;
        r.p1 = bop3<kSelect>(nt1, n.s0, n.s1);
        r.p2 = n.s2 | nt1;
        r.und = bop3<0x04>(n.s2, nt1, n.s1) | ~some;  // n_t = 1: n_s < 2
    } else {
        const uint64_t nt2 = bop3<kNeNe>(w, above, below);
        r.p0 = n.s0;
        r.p1 = n.s1 | nt2;
        if (regime == 1) {  // n_t = 0: n_s; n_t = 1: 4 + n_s; n_t = 2: 6
            asm volatile("");
            r.p2 = some;
            r.und = bop3<0x0B>(n.s2, some, bop3<0x07>(n.s1, nt2, n.s0));
        } else {            // n_t = 0: 4 + n_s; n_t = 1: n_s; n_t = 2: 2 + n_s
            r.p2 = ~some;
            r.und = bop3<0x1F>(n.s1, n.s0, some) & ~n.s2;
        }
    }
    return r;
}


// Where colour-c word `idx` of a slot has its neighbourhood, and its
// couplings.  Colour-c words of a slot are numbered plane by plane, row by
// row: idx = tau*(L*L/2) + y*(L/2) + xh, x = 2*xh + ((c + y + tau) & 1).
struct WordSite {
    uint32_t s, xp, xm, yp, ym, above, below;  // word indices in the slot
    uint32_t flip;                             // bit 0 / 1: above / below lies across the ends
    uint64_t jxp, jxm, jyp, jym;
};
template <bool kGlobal>
__device__ __forceinline__ WordSite locate_word(const GroupDev& G, const uint64_t* __restrict__ Jx,
                                                const uint64_t* __restrict__ Jy, uint32_t colour,
                                                uint32_t idx) {
    const uint32_t L = G.L;
    const uint32_t P = L * L;
    const uint32_t tau = fast_div(idx, G.div_half_plane);
    const uint32_t rem = idx - tau * (P >> 1);
    const uint32_t y = fast_div(rem, G.div_half_row);
    const uint32_t x = 2 * (rem - y * (L >> 1)) + ((colour + y + tau) & 1u);
    const uint32_t xp = (x + 1 == L) ? 0 : x + 1;
    const uint32_t xm = (x == 0) ? L - 1 : x - 1;
    const uint32_t yp = (y + 1 == L) ? 0 : y + 1;
    const uint32_t ym = (y == 0) ? L - 1 : y - 1;
    const uint32_t tp = (tau + 1 == G.Ltau) ? 0 : tau + 1;
    const uint32_t tm = (tau == 0) ? G.Ltau - 1 : tau - 1;
    const uint32_t row = y * L;
    const uint32_t plane = tau * P;
    WordSite r;
    r.s = plane + row + x;
    r.xp = plane + row + xp;
    r.xm = plane + row + xm;
    r.yp = plane + yp * L + x;
    r.ym = plane + ym * L + x;
    r.above = tp * P + row + x;
    r.below = tm * P + row + x;
    r.flip = (tp == 0 ? 1u : 0u) | (tau == 0 ? 2u : 0u);
    r.jxp = load64<kGlobal>(Jx, row + x);
    r.jxm = load64<kGlobal>(Jx, row + xm);  // the -x bond is the +x bond of x-1
    r.jyp = load64<kGlobal>(Jy, row + x);
    r.jym = load64<kGlobal>(Jy, ym * L + x);
    return r;
}

template <bool kGlobal>
__device__ __forceinline__ Word load_word(const GroupDev& G, const uint64_t* __restrict__ S,
                                          uint32_t regime, const WordSite& at) {
    const uint64_t w = load64<kGlobal>(S, at.s);
    const SpaceCount n =
        count_space(w, load64<kGlobal>(S, at.xp), load64<kGlobal>(S, at.xm),
                    load64<kGlobal>(S, at.yp), load64<kGlobal>(S, at.ym), at.jxp, at.jxm, at.jyp,
                    at.jym);
    uint64_t above = load64<kGlobal>(S, at.above);
    uint64_t below = load64<kGlobal>(S, at.below);
    // on an antiperiodic prism the bond that wraps round tau counts with the
    // opposite sign, which is the neighbour's word inverted
    if (G.anti) {
        asm volatile("");  // a block-uniform branch: periodic groups skip this
        if (at.flip & 1u) above = ~above;
        if (at.flip & 2u) below = ~below;
    }
    return class_code(regime, at.s, w, n, above, below);
}

// Threshold plane T of one level: bit j = the level's threshold bit of lane
// j's class, a function of the three code planes and so one v_bitop3 per
// 32-lane half.  That instruction takes its truth table as an immediate
// while the table differs from slot to slot and level to level, so there is
// one handler per table (128: code 7 does not occur) and the level jumps to
// its own: the two operations and a branch to the end, kHandlerBytes apart.
// Combining one-hot class masks under uniform branches instead took seven
// vector and fourteen scalar instructions a level and held fourteen registers
// of masks: 3089 vector instructions a wave of eight words and 5.6 waves a
// SIMD, now 2432 and 7.5, 783 -> 621 us a pass on 2 x 48 slots of 24 x 24 x
// 2048.  (Handlers that also hold the comparison, 64 bytes each, took 3 %
// longer: more instruction fetches.)  `entry`: byte offset of the handler from
// the instruction after s_getpc, as the host stores it per slot and level
// (level_entry); nothing else may be stored there.  The mask keeps the jump
// within the handlers and the three instructions before them, where offsets 0,
// 4 and 8 would jump for ever: a table that was never set is not run (the
// host refuses sweeps before every ladder is set).  (An offset that lands on
// a handler whatever the entry costs two more scalar instructions a Philox
// block, 1 to 2 % on small launches.)
__device__ __forceinline__ uint64_t threshold_plane(uint32_t entry, const Word& r) {
    static_assert(kHandlerBytes == 32 && kHandlerSkip == 12, "handlers below are laid out so");
    uint32_t T_lo, T_hi;
    asm("s_getpc_b64 vcc\n"
        "s_add_u32 vcc_lo, vcc_lo, %[e]\n"
        "s_addc_u32 vcc_hi, vcc_hi, 0\n"
        "s_setpc_b64 vcc\n"
        ".set .Lqsg_t%=, 0\n"
        ".rept 128\n"
        "v_bitop3_b32 %[tl], %[cl], %[bl], %[al] bitop3:.Lqsg_t%=\n"
        "v_bitop3_b32 %[th], %[ch], %[bh], %[ah] bitop3:.Lqsg_t%=\n"
        "s_branch .Lqsg_end%=\n"
        "s_nop 0\n"
        "s_nop 0\n"
        "s_nop 0\n"
        ".set .Lqsg_t%=, .Lqsg_t%= + 1\n"
        ".endr\n"
        ".Lqsg_end%=:\n"
        : [tl] "=&v"(T_lo), [th] "=&v"(T_hi)
        : [e] "s"(entry & kEntryMask), [al] "v"((uint32_t)r.p0), [ah] "v"((uint32_t)(r.p0 >> 32)),
          [bl] "v"((uint32_t)r.p1), [bh] "v"((uint32_t)(r.p1 >> 32)), [cl] "v"((uint32_t)r.p2),
          [ch] "v"((uint32_t)(r.p2 >> 32))
        : "vcc", "scc");
    return lo_hi(T_lo, T_hi);
}

// Compare the lanes' bit-sliced Philox numbers with their class thresholds,
// most significant level first, for blocks q0 <= q < q1 while any lane of
// the wave is undecided.  Block q (counter (s, t, g<<4 | q, gid)) carries
// levels 2q and 2q+1.  Per level, on each 32-bit half, with T the plane of
// the lanes' threshold bits and W the level of the random numbers:
//   acc = und ? T : acc   (a lane decided here has T != W: accepted iff T = 1)
//   und &= ~(T ^ W)       (still equal so far).
// So acc holds the decision of every lane once it has left und; on lanes
// still in und it is meaningless.
__device__ __forceinline__ void compare_levels(const GroupDev& G, uint32_t g, uint32_t t,
                                               const uint32_t* entries, const Word& r, uint32_t q0,
                                               uint32_t q1, uint64_t& acc, uint64_t& und) {
    // the slot's handler entries (two levels to a word), read through the
    // constant address space: block-uniform scalar loads (the table is not
    // written during a launch)
    typedef const uint32_t __attribute__((address_space(4)))* ConstU32;
    const ConstU32 en = (ConstU32)(entries);
    const PhiloxSite ps = philox_site(r.s, G.gid, G.key1);
#pragma unroll 1
    for (uint32_t q = q0; q < q1; ++q) {
        if (!__any(und != 0)) break;  // every lane of the wave decided
        const uint32_t e = en[q];
        const uint4 o = philox_block(ps, t, (g << 4) | q, G.key0, G.key1);
        uint64_t T = threshold_plane(e, r);
        acc = bop3<kSelect>(und, T, acc);
        und = bop3<kAndXnor>(und, T, lo_hi(o.x, o.y));
        T = threshold_plane(e >> 16, r);
        acc = bop3<kSelect>(und, T, acc);
        und = bop3<kAndXnor>(und, T, lo_hi(o.z, o.w));
    }
}

// Queue a word: w with the lanes accepted so far flipped.
__device__ __forceinline__ void push_word(SweepQueue& Q, uint32_t k, const Word& r, uint64_t w,
                                          uint64_t und) {
    Q.s[k] = r.s;
    Q.w[k] = w;
    Q.p0[k] = r.p0;
    Q.p1[k] = r.p1;
    Q.p2[k] = r.p2;
    Q.und[k] = und;
}

__device__ __forceinline__ Word pop_word(const SweepQueue& Q, uint32_t k) {
    return {Q.s[k], Q.w[k], Q.p0[k], Q.p1[k], Q.p2[k], Q.und[k]};
}

// The colour-pass update of one word per thread of the block: the first
// G.q_split Philox blocks of levels for every word; then, while the words
// with undecided lanes fill more than one wave, they are packed into the
// first waves of the block and given one more block; the last ones (at most
// one wave) are finished there.  Far fewer waves run the long tail of
// levels.  Every thread of the block calls this (it synchronises); `valid`
// is false for threads without a word (r is then unused).  Packing counters:
// one pair per call parity (see SweepQueue); within a call, round j writes
// counter j & 1, which round j - 1 cleared after every thread had read its
// previous value.
__device__ __forceinline__ void sweep_words(const GroupDev& G, uint64_t* __restrict__ S, uint32_t g,
                                            uint32_t t, const Word& r, bool valid, SweepQueue& Q,
                                            uint32_t parity) {
    const uint32_t* entries = G.thr + g * kThrStride + kLevelEntries;
    uint32_t* cnt = Q.count + 2 * (parity & 1u);
    if (threadIdx.x == 0) {
        cnt[0] = 0;
        cnt[1] = 0;
    }
    __syncthreads();
    if (valid) {
        uint64_t acc = ~r.und;  // lanes outside the seven classes: dE <= 0, accepted
        uint64_t und = r.und;
        compare_levels(G, g, t, entries, r, 0, G.q_split, acc, und);
        const uint64_t w = bop3<kXorAndNot>(r.w, acc, und);
        if (und != 0)
            push_word(Q, atomicAdd(&cnt[0], 1u), r, w, und);
        else
            store64<true>(S, r.s, w);
    }
    __syncthreads();
    uint32_t n = __builtin_amdgcn_readfirstlane(cnt[0]);
    uint32_t q = G.q_split;
#pragma unroll 1
    for (uint32_t j = 1; n != 0; ++j) {
        // the last words are finished where they sit in the queue: all 32
        // bits, and a lane equal on every one of them has r == thr, accepted
        const bool last = n <= kWaveSize || q + 1 >= 16;
        const uint32_t q1 = last ? 16 : q + 1;
        const bool have = threadIdx.x < n;
        Word e;
        if (have) e = pop_word(Q, threadIdx.x);
        if (!last) {
            __syncthreads();  // every entry and count read before any is rewritten
            if (threadIdx.x == 0) cnt[(j + 1) & 1u] = 0;
        }
        if (have) {
            uint64_t acc = 0, und = e.und;
            compare_levels(G, g, t, entries, e, q, q1, acc, und);
            const uint64_t w = bop3<kXorAndNot>(e.w, acc, und);
            if (last)
                store64<true>(S, e.s, w ^ und);
            else if (und != 0)
                push_word(Q, atomicAdd(&cnt[j & 1u], 1u), e, w, und);
            else
                store64<true>(S, e.s, w);
        }
        if (last) break;
        __syncthreads();
        n = __builtin_amdgcn_readfirstlane(cnt[j & 1u]);
        q = q1;
    }
}

// Column walk: thread `item` of a slot owns column (x, y) = item mod L^2 of
// tau tile item / L^2 (G.tile planes, tile * G.tile ... + G.tile - 1); its
// colour-c sites there are tau = tau0 + par, tau0 + par + 2, ..., with
// par = (c + x + y) & 1, one per step.  Offsets of the centre and its four
// space neighbours are fixed for the walk and the slot base advances by two
// planes per step (a block-uniform address on the scalar unit), the four
// couplings are loaded once into the thread's LDS slot (re-read from global
// memory every step, they cost 5 % of the pass), and the word below the
// centre is the previous step's word above it, so a step costs six loads and
// no index arithmetic.
// Only the first step's lower neighbour and the last step's upper one can
// wrap round tau.
__device__ __forceinline__ uint64_t load_at(const uint64_t* base, uint32_t byte_off) {
    return *(const uint64_t __attribute__((address_space(1)))*)((const GlobalByte*)base + byte_off);
}

// A block-uniform pointer read back through the scalar unit: the compiler
// then forms each address as this scalar base plus a 32-bit offset inside
// the loop instead of keeping 64-bit per-thread addresses live across it.
template <typename T>
__device__ __forceinline__ T* scalar_ptr(T* p) {
    const uint64_t v = (uint64_t)(uintptr_t)p;
    const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)v);
    const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)(v >> 32));
    return (T*)(uintptr_t)lo_hi(lo, hi);
}

__device__ __forceinline__ void walk_block(const GroupDev& G, uint64_t* __restrict__ S, uint32_t g,
                                           uint32_t colour, uint32_t t, uint32_t item,
                                           uint32_t n_items, SweepQueue& Q,
                                           WalkCouplings& J) {
    const bool valid = item < n_items;
    const uint32_t regime = __builtin_amdgcn_readfirstlane(G.thr[g * kThrStride + 15]);
    const uint32_t L = G.L, P = L * L, Ltau = G.Ltau;
    const uint32_t steps = G.tile >> 1;
    uint32_t tile = 0, col = 0;
    if (valid) {
        tile = fast_div(item, G.div_plane);
        col = item - tile * P;
    }
    const uint32_t y = fast_div(col, G.div_row);
    const uint32_t x = col - y * L;
    const uint32_t xp = (x + 1 == L) ? 0 : x + 1;
    const uint32_t xm = (x == 0) ? L - 1 : x - 1;
    const uint32_t yp = (y + 1 == L) ? 0 : y + 1;
    const uint32_t ym = (y == 0) ? L - 1 : y - 1;
    const uint32_t row = y * L;
    const uint32_t tau0 = tile * G.tile + ((colour + x + y) & 1u);
    const uint32_t plane0 = tau0 * P;
    // byte offsets from the step's base S + 2 k P (k = step)
    uint32_t o_c = (plane0 + row + x) * 8u;
    uint32_t o_xp = (plane0 + row + xp) * 8u, o_xm = (plane0 + row + xm) * 8u;
    uint32_t o_yp = (plane0 + yp * L + x) * 8u, o_ym = (plane0 + ym * L + x) * 8u;
    uint32_t o_tp = o_c + P * 8u;
    const uint32_t j_c = (row + x) * 8u, j_xm = (row + xm) * 8u, j_ym = (ym * L + x) * 8u;
    uint64_t below = 0;
    if (valid) {
        if (tau0 == 0) {  // the bond round tau: slice Ltau-1, sign flipped if antiperiodic
            below = load64<true>(S, (Ltau - 1) * P + row + x);
            if (G.anti) below = ~below;
        } else {
            below = load_at(S, o_c - P * 8u);
        }
    }
    const uint32_t site0 = plane0 + row + x;
    const uint64_t* S0 = scalar_ptr(S);
    const uint64_t* Jx = scalar_ptr(G.Jx);
    const uint64_t* Jy = scalar_ptr(G.Jy);
    const uint32_t i = threadIdx.x;
    if (valid) {
        J.xp[i] = load_at(Jx, j_c);
        J.xm[i] = load_at(Jx, j_xm);  // the -x bond is the +x bond of x-1
        J.yp[i] = load_at(Jy, j_c);
        J.ym[i] = load_at(Jy, j_ym);
    }
#pragma unroll 1
    for (uint32_t k = 0; k < steps; ++k) {
        const uint64_t* Sk = S0 + (size_t)k * 2 * P;
        // the offsets stay 32-bit values in the loop (scalar base + 32-bit
        // offset addressing), not 64-bit addresses hoisted out of it
        asm volatile("" : "+v"(o_c), "+v"(o_xp), "+v"(o_xm), "+v"(o_yp), "+v"(o_ym), "+v"(o_tp));
        Word r;
        if (valid) {
            const uint64_t w = load_at(Sk, o_c);
            uint64_t above;
            if (k + 1 == steps && tau0 + 2 * k + 1 == Ltau) {  // top slice: wraps to slice 0
                above = load64<true>(S, row + x);
                if (G.anti) above = ~above;
            } else {
                above = load_at(Sk, o_tp);
            }
            const SpaceCount n = count_space(w, load_at(Sk, o_xp), load_at(Sk, o_xm),
                                             load_at(Sk, o_yp), load_at(Sk, o_ym), J.xp[i],
                                             J.xm[i], J.yp[i], J.ym[i]);
            r = class_code(regime, site0 + 2 * k * P, w, n, above, below);
            below = above;
        }
        sweep_words(G, S, g, t, r, valid, Q, k);
    }
}

// Blocks are dealt to the eight XCDs round-robin (block b runs on XCD b % 8).
// Renumber them so that every XCD receives one contiguous run of logical
// blocks: neighbouring tau-planes then meet in the same L2.  A bijection of
// [0, n); only the speed depends on the dispatch order.  `backwards` runs
// each XCD through its blocks from the last to the first: the blue pass does,
// so that it begins with the words the red pass left in the caches (3 % less
// time per pass on ensembles of 0.5 to 0.9 GB).
__device__ __forceinline__ uint32_t xcd_contiguous(uint32_t b, uint32_t n, bool backwards = false) {
    constexpr uint32_t kXcd = 8;
    const uint32_t q = n / kXcd, r = n % kXcd;
    const uint32_t x = b % kXcd;
    uint32_t i = b / kXcd;
    if (backwards) i = q + (x < r ? 1 : 0) - 1 - i;
    return x < r ? x * (q + 1) + i : r * (q + 1) + (x - r) * q + i;
}

__global__ void __launch_bounds__(kSweepBlock)
k_half_sweep(const GroupDev G, uint32_t colour, const uint32_t* __restrict__ ctr, uint32_t t_add) {
    __shared__ SweepQueue Q;
    __shared__ WalkCouplings J;
    const uint32_t t = __builtin_amdgcn_readfirstlane(ctr[0] + t_add);
    const uint32_t b = xcd_contiguous(blockIdx.y * gridDim.x + blockIdx.x, gridDim.x * gridDim.y,
                                      colour != 0);
    const uint32_t g = fast_div(b, G.div_blocks);  // b / gridDim.x on the scalar unit
    const uint32_t item = (b - g * gridDim.x) * kSweepBlock + threadIdx.x;
    walk_block(G, G.spins + (size_t)g * G.V, g, colour, t, item, G.V >> __builtin_ctz(G.tile), Q,
               J);
}

__device__ __forceinline__ uint32_t find_group(const uint32_t* __restrict__ prefix,
                                               uint32_t n_groups, uint32_t b) {
    uint32_t lo = 0, hi = n_groups;
    while (hi - lo > 1) {
        const uint32_t mid = (lo + hi) >> 1;
        if (prefix[mid] <= b) lo = mid; else hi = mid;
    }
    return lo;
}

// Record of group gi.  For groups of one shape (kSameShape: the plan's
// same_shape, chosen at launch so that each instantiation has one path) it
// is the kernel argument's copy with the pointers moved to group gi and the
// group's own Philox identity: no load stands between the block's start and
// its first address computation (the three identity words are needed only
// later).  Otherwise the record is read from memory.
template <typename T>
__device__ __forceinline__ T* advance(T* p, uint64_t bytes) {
    return (T*)((char*)p + bytes);
}
template <bool kSameShape>
__device__ __forceinline__ GroupDev group_record(const BatchPlan& p, uint32_t gi) {
    if (!kSameShape) return uniform_record(p.groups + gi);
    GroupDev G = p.first;
    const uint64_t d = (uint64_t)gi * p.stride;
    G.spins = advance(G.spins, d);
    G.Jx = advance(G.Jx, d);
    G.Jy = advance(G.Jy, d);
    G.jseed = advance(G.jseed, d);
    G.thr = advance(G.thr, d);
    G.sw_thr = advance(G.sw_thr, d);
    G.sw_len = advance(G.sw_len, d);
    G.sw_eq = advance(G.sw_eq, d);
    G.cnt = advance(G.cnt, d);
    G.E = advance(G.E, d);
    G.walker = advance(G.walker, d);
    G.rt = advance(G.rt, d);
    G.acc = advance(G.acc, d);
    G.swaplog = advance(G.swaplog, d);
    G.sums = advance(G.sums, d);
    G.lastmask = advance(G.lastmask, d);
    G.meas = advance(G.meas, d);
    G.hist = advance(G.hist, d);
    const GroupDev* __restrict__ r = p.groups + gi;
    G.gid = __builtin_amdgcn_readfirstlane(r->gid);
    G.key0 = __builtin_amdgcn_readfirstlane(r->key0);
    G.key1 = __builtin_amdgcn_readfirstlane(r->key1);
    return G;
}

// Group of block b of a batched launch and the block's index within that
// group.  Groups of one size (the usual ensemble) take one scalar division;
// otherwise one load from the plan's block map where it has one, else a
// binary search of the prefix sums (a chain of dependent scalar loads that
// delays every block's first spin load).  kSameShape: the plan's groups
// share one shape, so they have equal block counts and only the division is
// compiled in.
struct BlockPlace {
    uint32_t gi, local;
};
template <bool kSameShape>
__device__ __forceinline__ BlockPlace locate(const BatchPlan& p, uint32_t b) {
    if (kSameShape || p.per_group) {
        const uint32_t gi = fast_div(b, p.span);
        return {gi, b - gi * p.per_group};
    }
    if (p.block_map) {
        const BlockEntry e = p.block_map[b];
        return {(uint32_t)__builtin_amdgcn_readfirstlane(e.gi),
                (uint32_t)__builtin_amdgcn_readfirstlane(e.local)};
    }
    const uint32_t gi = find_group(p.prefix, p.n_groups, b);
    return {gi, b - p.prefix[gi]};
}

template <bool kSameShape>
__global__ void __launch_bounds__(kSweepBlock)
k_half_sweep_batched(const BatchPlan plan, uint32_t colour, const uint32_t* __restrict__ ctr,
                     uint32_t t_add) {
    __shared__ SweepQueue Q;
    __shared__ WalkCouplings J;
    const uint32_t t = __builtin_amdgcn_readfirstlane(ctr[0] + t_add);
    const uint32_t b = xcd_contiguous(blockIdx.x, gridDim.x, colour != 0);
    const BlockPlace at = locate<kSameShape>(plan, b);
    const GroupDev G = group_record<kSameShape>(plan, at.gi);
    const uint32_t local = __builtin_amdgcn_readfirstlane(at.local);
    const uint32_t nb = sweep_blocks_per_slot(G.V, G.tile);
    const uint32_t g = fast_div(local, G.div_blocks);  // local / nb on the scalar unit
    const uint32_t item = (local - g * nb) * kSweepBlock + threadIdx.x;
    walk_block(G, G.spins + (size_t)g * G.V, g, colour, t, item, G.V >> __builtin_ctz(G.tile), Q,
               J);
}

// ---------------------------------------------------------------------------
// Fused sweeps: one block owns one slot for `n_sweeps` sweeps (no other
// block touches it before the PT step), so colour passes are separated by
// block barriers only and all sweeps of a PT chunk are one launch.  One word
// per thread and round.  The slots run from LDS (kLds: spins, then the
// couplings, copied in, and the spins back), or from global memory where the
// launch's largest slot does not fit.
//
// What bounds it: vector issue of the one CU a slot is on (3.4 us per pass of
// 1024 words; 16 waves of 515 instructions are 3.7 us at 2.2 GHz), below a
// few hundred words the latency of one word's comparison (2 us).  So every
// wave takes its words to the end by itself: packing the words still
// undecided, as the colour pass does, saves a fifth of the comparisons but
// costs barriers and LDS traffic that one block per CU cannot hide (4.8 us),
// and one Philox block per wave of a shared word, or two at a time, no less
// (4.9, 4.0).  Where the block has a thread for every word of a colour the
// neighbourhoods are found once (3.9 us if found in every pass).  With 256
// threads, packing and the couplings in global memory a pass took 12.4 us;
// the colour passes of a graph take 5.7 each on so few words.
// ---------------------------------------------------------------------------
template <bool kGlobal>
__device__ __forceinline__ void update_word(const GroupDev& G, uint64_t* __restrict__ S,
                                            uint32_t regime, uint32_t g, uint32_t t,
                                            const WordSite& at) {
    const Word r = load_word<kGlobal>(G, S, regime, at);
    uint64_t acc = ~r.und, und = r.und;  // lanes outside the seven classes: dE <= 0, accepted
    compare_levels(G, g, t, G.thr + g * kThrStride + kLevelEntries, r, 0, 16, acc, und);
    // a lane equal on all 32 bits has r == thr, accepted
    store64<kGlobal>(S, r.s, bop3<kXorAndNot>(r.w, acc, und) ^ und);
}

template <bool kLds>
__global__ void __launch_bounds__(kFusedBlock, 8)
k_chunk_fused(const BatchPlan slots, const uint32_t* __restrict__ ctr, uint32_t n_sweeps) {
    extern __shared__ uint64_t lds_words[];
    const BlockPlace at = locate<false>(slots, blockIdx.x);
    const GroupDev G = group_record<false>(slots, at.gi);
    const uint32_t g = __builtin_amdgcn_readfirstlane(at.local);
    const uint32_t V = G.V, half = V >> 1, P = G.L * G.L;
    uint64_t* Sg = G.spins + (size_t)g * V;
    const uint32_t regime = __builtin_amdgcn_readfirstlane(G.thr[g * kThrStride + 15]);
    if (kLds) {
        for (uint32_t i = threadIdx.x; i < V; i += blockDim.x) lds_words[i] = Sg[i];
        for (uint32_t i = threadIdx.x; i < P; i += blockDim.x) {
            lds_words[V + i] = G.Jx[i];
            lds_words[V + P + i] = G.Jy[i];
        }
        __syncthreads();
    }
    const uint32_t t0 = __builtin_amdgcn_readfirstlane(ctr[0]);
    uint64_t* S = kLds ? lds_words : Sg;
    const uint64_t* Jx = kLds ? lds_words + V : G.Jx;
    const uint64_t* Jy = kLds ? lds_words + V + P : G.Jy;
    if (kLds && half <= blockDim.x) {  // a thread's two words are the same in every sweep
        const uint32_t idx = threadIdx.x;
        WordSite red{}, blue{};
        if (idx < half) {
            red = locate_word<!kLds>(G, Jx, Jy, 0, idx);
            blue = locate_word<!kLds>(G, Jx, Jy, 1, idx);
        }
#pragma unroll 1
        for (uint32_t it = 0; it < n_sweeps; ++it) {
            if (idx < half) update_word<!kLds>(G, S, regime, g, t0 + it, red);
            __syncthreads();  // the next colour reads what this one wrote
            if (idx < half) update_word<!kLds>(G, S, regime, g, t0 + it, blue);
            __syncthreads();
        }
    } else {
#pragma unroll 1
        for (uint32_t pass = 0; pass < 2 * n_sweeps; ++pass) {
#pragma unroll 1
            for (uint32_t idx = threadIdx.x; idx < half; idx += blockDim.x)
                update_word<!kLds>(G, S, regime, g, t0 + (pass >> 1),
                                   locate_word<!kLds>(G, Jx, Jy, pass & 1u, idx));
            __syncthreads();
        }
    }
    if (kLds)
        for (uint32_t i = threadIdx.x; i < V; i += blockDim.x) Sg[i] = lds_words[i];
}

// ---------------------------------------------------------------------------
// Energy / overlap pass: per slot and lane, the number of unsatisfied space
// bonds and time bonds (each bond counted once, from its lower endpoint),
// and per lane pair (2p, 2p+1) the number of sites where they differ.
// Each thread adds its words into bit-sliced vertical counters; each wave
// then turns counters into per-lane totals (a bit transpose across the wave
// and popcounts) and adds them to the slot's counters with integer atomics
// (order-independent, exact).
// ---------------------------------------------------------------------------
// Bit-sliced per-lane counter: value = ones + 2 twos + 4 fours + 8 * (hi as
// a binary number).  Planes are added eight at a time with carry-save adders
// (Harley-Seal): seven adders, then the binary part rippled once.
// Binary planes a LaneCounter needs above ones/twos/fours to hold `max`.
constexpr int counter_planes(int max) {
    int nh = 0;
    while ((8 << nh) - 1 < max) ++nh;
    return nh;
}

template <int NH>
struct LaneCounter {
    uint64_t ones = 0, twos = 0, fours = 0;
    uint64_t hi[NH] = {};
};

// carry-save adder: (h, l) with a + b + c = 2h + l per lane
__device__ __forceinline__ void csa(uint64_t& h, uint64_t& l, uint64_t a, uint64_t b, uint64_t c) {
    const uint32_t alo = (uint32_t)a, blo = (uint32_t)b, clo = (uint32_t)c;
    const uint32_t ahi = (uint32_t)(a >> 32), bhi = (uint32_t)(b >> 32), chi = (uint32_t)(c >> 32);
    l = lo_hi(__builtin_amdgcn_bitop3_b32(alo, blo, clo, 0x96),
              __builtin_amdgcn_bitop3_b32(ahi, bhi, chi, 0x96));  // a ^ b ^ c
    h = lo_hi(__builtin_amdgcn_bitop3_b32(alo, blo, clo, 0xE8),
              __builtin_amdgcn_bitop3_b32(ahi, bhi, chi, 0xE8));  // majority
}

// Four words into `ones` and `twos`; what they carry into the fours.
template <int NH>
__device__ __forceinline__ uint64_t add4(LaneCounter<NH>& c, const uint64_t (&x)[4]) {
    uint64_t twosA, twosB, fours;
    csa(twosA, c.ones, c.ones, x[0], x[1]);
    csa(twosB, c.ones, c.ones, x[2], x[3]);
    csa(fours, c.twos, c.twos, twosA, twosB);
    return fours;
}

// The carries of two such additions.
template <int NH>
__device__ __forceinline__ void add_fours(LaneCounter<NH>& c, uint64_t a, uint64_t b) {
    uint64_t eights;
    csa(eights, c.fours, c.fours, a, b);
#pragma unroll
    for (int i = 0; i < NH; ++i) {
        const uint64_t carry = c.hi[i] & eights;
        c.hi[i] ^= eights;
        eights = carry;
    }
}

// 64 x 64 bit transpose across the wave: afterwards thread t holds, in bit
// b, bit t of thread b's word.  Stage k exchanges with thread t ^ 2^k the
// bits whose index differs from t in bit k (swapping bit k of the thread
// index with bit k of the bit index); the six stages commute.  Stage 5
// swaps the roles of the two 32-bit halves: a thread sends its partner the
// half the partner keeps and takes one half back.  Stages 0-4 stay inside
// each half: a thread keeps its bits on one side of bit k (mask K) and takes
// the partner's other side, rotated into place by one v_alignbit (right by
// 2^k if it keeps the upper side, else by 32 - 2^k), then one v_bitop3
// merges the two.
__device__ __forceinline__ uint64_t wave_transpose(uint64_t x) {
    const uint32_t t = threadIdx.x & 63u;
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
        lo = BITOP3(keep, lo, __builtin_amdgcn_alignbit(ylo, ylo, rot), kSelect);
        hi = BITOP3(keep, hi, __builtin_amdgcn_alignbit(yhi, yhi, rot), kSelect);
    }
    return lo_hi(lo, hi);
}

// Per-lane totals over the wave's 64 threads of a bit-sliced counter: thread
// t gets the total of lane t.
template <int NH>
__device__ __forceinline__ uint32_t lane_total(const LaneCounter<NH>& c) {
    uint32_t tot = (uint32_t)__popcll(wave_transpose(c.ones)) +
                   ((uint32_t)__popcll(wave_transpose(c.twos)) << 1) +
                   ((uint32_t)__popcll(wave_transpose(c.fours)) << 2);
#pragma unroll
    for (int i = 0; i < NH; ++i) tot += (uint32_t)__popcll(wave_transpose(c.hi[i])) << (3 + i);
    return tot;
}

// Column walk: thread `item` of slot g owns column (x, y) = item mod L^2 of
// tau tile item / L^2 and walks it bottom to top.  The slot's `tiles` tiles
// have planes = ceil(Ltau / tiles) planes, the first tiles * planes - Ltau
// of them one less.  Each bond is counted once, from its lower endpoint: per
// word the +x and +y neighbours in the same plane and the word above, which
// is the next step's centre, so a step costs three loads; the offsets are
// fixed for the walk and the slot base advances one plane per step.  Only
// the last tile's last bond can wrap round tau.
//
// The walk runs in batches of kEnergyBatch steps, software-pipelined: the
// loads of the next batch are issued before the current batch is counted,
// so every wave keeps loads in flight while it adds.  For that the loads of
// a batch take no branch (the compiler would otherwise wait for every load
// in flight before counting): steps past the tile's end re-read its last
// plane and are not counted, the wrapping bond's word comes through a
// selected offset, and its antiperiodic sign is applied when counting.  A
// short tile's step planes-1 lies in the tile above it (the last tile is
// never short), so it is read like any other and masked out.
//
// What bounds it: on a full chip the reads of the spins (67 M words take 160
// us after the colour passes of a chunk and 182 after an exchange pass, 3.4
// and 2.9 TB/s; 113 M after an exchange pass 257 us, 3.5 TB/s: a third fewer
// instructions in the adds changed neither); on few words the transposes at
// the end of every wave (16 to 22 of them, as many instructions as 16 planes)
// against too few waves, and where few slots are large the waves' atomics on
// one set of counters: energy_walks picks the depth.
constexpr int kEnergyBatch = 4;

struct EnergyBatch {
    uint64_t up[kEnergyBatch], xp[kEnergyBatch], yp[kEnergyBatch];
};

template <int kMaxPlanes>
__device__ __forceinline__ void energy_walk(const GroupDev& G, uint32_t g, uint32_t item,
                                            const EnergyWalks W, int32_t* __restrict__ cnt) {
    const uint32_t L = G.L, P = L * L, planes = W.planes;
    const uint32_t n_items = P * W.tiles;
    // a wave without a column (the tail of a slot's last block) has nothing
    // to add: it leaves before the cross-lane transposes
    if (__builtin_amdgcn_readfirstlane(item) >= n_items) return;
    const uint64_t* __restrict__ S = G.spins + (size_t)g * G.V;
    // per thread and lane at most 2*kMaxPlanes unsatisfied space bonds and
    // kMaxPlanes time bonds or differing pairs
    LaneCounter<counter_planes(2 * kMaxPlanes)> Csp;
    LaneCounter<counter_planes(kMaxPlanes)> Ct, Cq;
    if (item < n_items) {
        const uint32_t tile = fast_div(item, G.div_plane);
        const uint32_t col = item - tile * P;
        const uint32_t y = fast_div(col, G.div_row);
        const uint32_t x = col - y * L;
        const uint32_t xp = (x + 1 == L) ? 0 : x + 1;
        const uint32_t yp = (y + 1 == L) ? 0 : y + 1;
        const uint32_t base = (tile * planes - min(tile, W.n_short)) * P;
        // byte offsets: o_xp, o_yp from the step's plane; up words from S
        uint32_t o_xp = (base + y * L + xp) * 8u, o_yp = (base + yp * L + x) * 8u;
        uint32_t o_up = (base + col + P) * 8u;
        const uint32_t o_wrap = col * 8u;  // slice 0, above the top slice
        const uint64_t jx = G.Jx[col], jy = G.Jy[col];
        const bool top = tile + 1 == W.tiles;  // the last bond wraps to slice 0
        const uint64_t flip = (top && G.anti) ? ~0ull : 0ull;  // antiperiodic wrap bond
        const uint32_t last = planes - 1;
        const uint64_t live = tile < W.n_short ? 0ull : ~0ull;  // step `last` belongs to the tile
        auto fetch = [&](uint32_t k0, EnergyBatch& B) {
            asm volatile("" : "+v"(o_up), "+v"(o_xp), "+v"(o_yp));  // 32-bit offsets in the loop
#pragma unroll
            for (int k = 0; k < kEnergyBatch; ++k) {
                const uint32_t kk = min(k0 + k, last);  // block-uniform
                const uint64_t* Sk = scalar_ptr(S + (size_t)kk * P);
                B.xp[k] = load_at(Sk, o_xp);
                B.yp[k] = load_at(Sk, o_yp);
                B.up[k] = load_at(S, (top && kk == last) ? o_wrap : o_up + kk * P * 8u);
            }
        };
        uint64_t w = load_at(S, (base + col) * 8u);
        // kGuard: some steps of the batch may lie past the tile's end
        // ct, cq: the batch's carries into the fours of Ct and Cq
        auto count = [&](auto guard, uint32_t k0, const EnergyBatch& B, uint64_t& ct, uint64_t& cq) {
            constexpr bool kGuard = decltype(guard)::value;
            uint64_t xs[kEnergyBatch], ys[kEnergyBatch], ts[kEnergyBatch], qs[kEnergyBatch];
#pragma unroll
            for (int k = 0; k < kEnergyBatch; ++k) {
                xs[k] = ys[k] = ts[k] = qs[k] = 0;
                if (!kGuard || k0 + k < planes) {  // block-uniform
                    const uint64_t up = B.up[k];
                    xs[k] = bop3<kXor3>(w, B.xp[k], jx);  // +x bond unsatisfied
                    ys[k] = bop3<kXor3>(w, B.yp[k], jy);  // +y bond unsatisfied
                    ts[k] = bop3<kXor3>(w, up, k0 + k == last ? flip : 0ull);  // +tau bond
                    // pair (2p, 2p+1) differs; pairs never straddle the halves
                    const uint32_t lo = (uint32_t)w, hi = (uint32_t)(w >> 32);
                    qs[k] = lo_hi(BITOP3(lo, lo >> 1, 0x55555555u, 0x28),
                                  BITOP3(hi, hi >> 1, 0x55555555u, 0x28));
                    w = up;
                    if (kGuard && k0 + k == last) {
                        xs[k] &= live;
                        ys[k] &= live;
                        ts[k] &= live;
                        qs[k] &= live;
                    }
                }
            }
            const uint64_t cx = add4(Csp, xs);
            add_fours(Csp, cx, add4(Csp, ys));
            ct = add4(Ct, ts);
            cq = add4(Cq, qs);
        };
        EnergyBatch b0, b1;
        uint64_t ct0, cq0, ct1, cq1;
        static_assert(2 * kEnergyBatch == 8, "walks_ahead");
        if (walks_ahead(W)) {
            // two batch buffers used in turn (no copies between them); the
            // last fetch re-reads the top plane and is not counted
            fetch(0, b0);
#pragma unroll 1
            for (uint32_t k0 = 0; k0 < planes; k0 += 2 * kEnergyBatch) {
                fetch(k0 + kEnergyBatch, b1);
                count(std::false_type{}, k0, b0, ct0, cq0);
                fetch(k0 + 2 * kEnergyBatch, b0);
                count(std::false_type{}, k0 + kEnergyBatch, b1, ct1, cq1);
                add_fours(Ct, ct0, ct1);
                add_fours(Cq, cq0, cq1);
            }
        } else {
#pragma unroll 1
            for (uint32_t k0 = 0; k0 < planes; k0 += kEnergyBatch) {
                fetch(k0, b0);
                count(std::true_type{}, k0, b0, ct0, cq0);
                add_fours(Ct, ct0, 0);
                add_fours(Cq, cq0, 0);
            }
        }
    }
    // every thread of the wave takes part in the transposes
    const uint32_t lane = threadIdx.x & 63u;
    const uint32_t my_sp = lane_total(Csp), my_t = lane_total(Ct);
    const uint32_t my_q = lane_total(Cq);  // pair p's total sits at lane 2p
    int32_t* __restrict__ c = cnt + g * kCntStride;
    if (my_sp) atomicAdd(&c[lane], (int32_t)my_sp);
    if (my_t) atomicAdd(&c[64 + lane], (int32_t)my_t);
    if (!(lane & 1u) && my_q) atomicAdd(&c[128 + (lane >> 1)], (int32_t)my_q);
}

template <int kMaxPlanes>
__global__ void __launch_bounds__(kEnergyBlock)
k_energy(const GroupDev G, int32_t* cnt, const EnergyWalks walks) {
    energy_walk<kMaxPlanes>(G, blockIdx.y, blockIdx.x * kEnergyBlock + threadIdx.x, walks, cnt);
}

template <int kMaxPlanes>
__global__ void __launch_bounds__(kEnergyBlock)
k_energy_batched(const BatchPlan plan, uint32_t reading) {
    const BlockPlace at = locate<false>(plan, blockIdx.x);
    const GroupDev G = group_record<false>(plan, at.gi);
    const uint32_t local = at.local;
    const uint32_t nb = energy_blocks_per_slot(G.L * G.L, G.ewalk.tiles);
    // block-uniform: keeps the slot's address arithmetic on the scalar unit
    const uint32_t g = __builtin_amdgcn_readfirstlane(local / nb);
    energy_walk<kMaxPlanes>(G, g, (local - g * nb) * kEnergyBlock + threadIdx.x, G.ewalk,
                            reading ? G.meas : G.cnt);
}

// ---------------------------------------------------------------------------
// Parallel tempering step of one group: one block, thread j of a wave = lane
// j.  In order: (1) the waves share the slots: each turns the pass counters
// of its slots into bond sums, adds them to the measurement sums, and works
// out what the pair (g, g+1) accepts; (2) the first wave visits the pairs g =
// 0..N-2 in order, `cur` being the configuration that currently sits at slot
// g (it may have arrived from g-1 in this step); (3) the waves share the
// slots again and write the new state.
//
// What bounds it: latency alone.  Only (2) is a chain, so everything that
// does not depend on the pairs before is moved out of it: a pair's random
// numbers, and its exchange table too, for the table falls with m and so
// "random number <= entry m" is "m <= most" with a `most` found beforehand
// (most_accepted).  The chain is left with LDS reads that can run ahead, one
// comparison and a ballot.  Per launch: 6.5 us for one group of 16 slots, 18.5
// for 64 of 32, 37 for two of 48 with long tables; one wave doing it all, with
// a table look-up and a Philox block in every link, took 23, 79 and 114.
// ---------------------------------------------------------------------------
struct PtShared {
    int32_t sp[kMaxSlots][64];     // space-bond sums
    int32_t e[kMaxSlots][64];      // what the exchange weighs: time bonds, or all
    uint32_t most[kMaxSlots][64];  // pair (g, g+1) accepts -D = 4m for m <= most
    uint8_t walker[kMaxSlots][64];
    uint8_t from[kMaxSlots][64];   // slot that slot g's new configuration comes from
};
constexpr uint32_t kAlways = 0xFFFFFFFFu;

// Entries of a falling table that are >= r (r > 0).  The entries are 2^32
// q^m rounded down, so the logarithms of r and of the first entry give the
// count to one or two; four entries around it settle it, or else a search of
// the table.
__device__ __forceinline__ uint32_t most_accepted(const uint32_t* __restrict__ thr, uint32_t len,
                                                  uint32_t r) {
    if (len == 0) return 0;
    constexpr float kUnit = 2.3283064365386963e-10f;  // 2^-32
    const float lq = log1pf(-(float)(0u - thr[0]) * kUnit);
    const float lr = r < 0x80000000u ? logf((float)r * kUnit) : log1pf(-(float)(0u - r) * kUnit);
    const uint32_t near = (uint32_t)fminf(fmaxf(lr / lq, 0.f), (float)len);
    const uint32_t base = near > 2 ? near - 2 : 0;
    uint32_t n = 0;
#pragma unroll
    for (uint32_t k = 0; k < 4; ++k) {
        const uint32_t t = thr[min(base + k, len - 1)];
        n += (base + k < len && t >= r) ? 1u : 0u;
    }
    if ((n > 0 || base == 0) && (n < 4 || base + 4 >= len)) return base + n;
    uint32_t lo = 0, hi = len;
    while (lo < hi) {
        const uint32_t mid = (lo + hi) >> 1;
        if (thr[mid] >= r)
            lo = mid + 1;
        else
            hi = mid;
    }
    return lo;
}

__device__ __forceinline__ void pt_group(const GroupDev& G, uint32_t p) {
    __shared__ PtShared sh;
    const uint32_t j = threadIdx.x & 63u;
    const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    constexpr uint32_t kWaves = kPtBlock / 64;
    const uint32_t N = G.N;
    const int32_t V = (int32_t)G.V;
    for (uint32_t g = wave; g < N; g += kWaves) {
        int32_t* __restrict__ c = G.cnt + g * kCntStride;
        int64_t* __restrict__ sm = G.sums + (size_t)g * kSumStride;
        const int32_t csp = c[j], ct = c[64 + j], cq = j < 32 ? c[128 + j] : 0;
        const int64_t s0 = sm[j], s1 = sm[64 + j];
        const int64_t s2 = j < 32 ? sm[128 + j] : 0, s3 = j < 32 ? sm[160 + j] : 0;
        const uint32_t w = G.walker[g * 64 + j];
        uint32_t most = 0;
        if (g + 1 < N) {
            const uint4 o = philox(make_uint4(j >> 2, p, (1u << 24) | g, G.gid), G.key0, G.key1);
            const uint32_t sel = j & 3u;
            const uint32_t r = sel == 0 ? o.x : sel == 1 ? o.y : sel == 2 ? o.z : o.w;
            most = G.sw_eq[g] || r == 0
                       ? kAlways
                       : most_accepted(G.sw_thr + (size_t)g * G.sw_cap, G.sw_len[g], r);
        }
        // |bsp| <= 2V and |bt| <= V with V <= 2^29: their sum fits 32 bits,
        // and the difference of two such sums fits 32 bits without a sign
        const int32_t bsp = 2 * V - 2 * csp;
        const int32_t bt = V - 2 * ct;
        sh.sp[g][j] = bsp;
        sh.e[g][j] = G.exch_all ? bsp + bt : bt;
        sh.most[g][j] = most;
        sh.walker[g][j] = (uint8_t)w;
        c[j] = 0;
        c[64 + j] = 0;
        sm[j] = s0 + bsp;
        sm[64 + j] = s1 + bt;
        if (j < 32) {
            const int64_t q = (int64_t)V - 2 * (int64_t)cq;
            c[128 + j] = 0;
            sm[128 + j] = s2 + q;
            sm[160 + j] = s3 + q * q;
        }
        // floor(u * bins / (V + 1)): both below 2^53 and the quotient, if not
        // whole, at least 2^-30 away from a whole number, so the rounded
        // quotient has the same floor
        const uint32_t u = (uint32_t)(V - bt) >> 1;
        const uint32_t bin = (uint32_t)(((double)u * kHistBins) / ((double)V + 1.0));
        atomicAdd(&G.hist[g * kHistBins + bin], 1u);
    }
    __syncthreads();
    if (wave == 0) {
        const uint64_t acc0 = j + 1 < N ? G.acc[j] : 0;
        int32_t cur = sh.e[0][j];
        uint32_t cur_from = 0;
        uint64_t my_mask = 0, any = 0;
        for (uint32_t g = 0; g + 1 < N; ++g) {
            const int32_t nx = sh.e[g + 1][j];
            const uint32_t most = sh.most[g][j];
            // D = nx - cur: accepted if D >= 0, else if m = -D / 4 <= most
            const uint32_t m = ((uint32_t)cur - (uint32_t)nx) >> 2;
            const bool accept = nx >= cur || m - 1u < most || most == kAlways;
            const uint64_t mask = __ballot((int)accept);
            // accepted: slot g takes the next configuration, cur moves up;
            // else cur stays at g and the next one becomes cur
            sh.from[g][j] = (uint8_t)(accept ? g + 1 : cur_from);
            cur = accept ? cur : nx;
            cur_from = accept ? cur_from : g + 1;
            my_mask = j == g ? mask : my_mask;
            any |= mask;
        }
        sh.from[N - 1][j] = (uint8_t)cur_from;
        if (j + 1 < N) {
            G.swaplog[(size_t)(p % G.log_cap) * (N - 1) + j] = my_mask;
            G.acc[j] = acc0 + (uint64_t)__popcll(my_mask);
            G.lastmask[j] = my_mask;
        }
        if (j == 0) G.lastmask[N - 1] = any ? 1ull : 0ull;
    }
    __syncthreads();
    // round trips 0 -> N-1 -> 0; this step ends at PT time p+1.  One slot
    // has no exchange partner and no pair of distinct end slots: its walkers
    // never move, and no round trip is counted.
    const uint32_t now = p + 1;
    if (wave == kWaves - 1 && N >= 2) {
        RoundTrip& r0 = G.rt[sh.walker[sh.from[0][j]][j] * 64 + j];
        if (r0.state == 2) {
            r0.count += 1;
            r0.sum += (uint64_t)(now - r0.t_last);
            r0.t_last = now;
            r0.state = 1;
        } else if (r0.state == 0) {
            r0.t_last = now;
            r0.state = 1;
        }
    }
    if (wave == kWaves - 2 && N >= 2) {  // another walker's record
        RoundTrip& rtop = G.rt[sh.walker[sh.from[N - 1][j]][j] * 64 + j];
        if (rtop.state == 1) rtop.state = 2;
    }
    for (uint32_t g = wave; g < N; g += kWaves) {
        const uint32_t f = sh.from[g][j];
        const int32_t bsp = sh.sp[f][j], e = sh.e[f][j];
        G.E[(g * 64 + j) * 2 + 0] = bsp;
        G.E[(g * 64 + j) * 2 + 1] = G.exch_all ? e - bsp : e;
        G.walker[g * 64 + j] = sh.walker[f][j];
    }
}

__global__ void __launch_bounds__(kPtBlock)
k_pt(const GroupDev G, const uint32_t* __restrict__ ctr) {
    pt_group(G, ctr[1]);
}

__global__ void __launch_bounds__(kPtBlock)
k_pt_batched(const GroupDev* __restrict__ groups, const uint32_t* __restrict__ ctr) {
    const GroupDev G = uniform_record(groups + blockIdx.x);
    pt_group(G, ctr[1]);
}

// Sweep and PT counters live on the device so that a captured graph can be
// replayed: every launch reads them and adds its own offset.
__device__ __forceinline__ void advance_counters(const Advance& a) {
    a.ctr[0] += a.dt;
    a.ctr[1] += a.dp;
}
__global__ void k_advance(const Advance a) {
    if (threadIdx.x == 0) advance_counters(a);
}

// ---------------------------------------------------------------------------
// Apply the accepted exchanges of the latest PT step to the spins: at every
// site, the pairs' masked bit exchanges in ascending order (each word read
// and written once).  On few sites the pass lasts as long as one site's
// chain: the slots' words are then loaded a batch ahead of the stores
// (kAhead), which the compiler may not reorder (4.3 us for 16 slots of 2048
// words, 7.0 with one load per link; 11.9 and 13.1 for 570 blocks).  Once the
// blocks fill the chip more than once it lasts as long as the copy of the
// spins, and one load per link is as fast or faster (172 us either way on 537
// MB, 321 against 337 on 906 MB).  The pass reads neither counter, and it is
// the last of a PT step: its first thread advances them, which saves the
// launch of its own that this took (4 us).
// ---------------------------------------------------------------------------
constexpr uint32_t kSwapBatch = 8;
constexpr uint32_t kSwapAheadBlocks = 2048;  // eight blocks on each of 256 CUs
template <bool kAhead>
__device__ __forceinline__ void swap_site(const GroupDev& G, uint32_t site) {
    constexpr uint32_t kBatch = kAhead ? kSwapBatch : 1;
    const uint32_t pairs = G.N - 1;
    uint64_t* S = G.spins + site;
    const size_t V = G.V;
    uint64_t cur = S[0];  // running content of slot g
    uint64_t orig = cur;  // what slot g held before this step
    for (uint32_t g0 = 0; g0 < pairs; g0 += kBatch) {
        uint64_t next[kBatch], mask[kBatch];
#pragma unroll
        for (uint32_t k = 0; k < kBatch; ++k) {
            const uint32_t g = min(g0 + k, pairs - 1);  // block-uniform
            next[k] = S[(size_t)(g + 1) * V];
            mask[k] = G.lastmask[g];
        }
#pragma unroll
        for (uint32_t k = 0; k < kBatch; ++k) {
            if (g0 + k >= pairs) break;
            const uint64_t d = (cur ^ next[k]) & mask[k];
            cur ^= d;
            if (cur != orig) S[(size_t)(g0 + k) * V] = cur;
            cur = next[k] ^ d;
            orig = next[k];
        }
    }
    if (cur != orig) S[(size_t)pairs * V] = cur;
}

template <bool kAhead>
__global__ void __launch_bounds__(kSwapBlock) k_swap_apply(const GroupDev G, const Advance adv) {
    if (adv.ctr && (blockIdx.x | threadIdx.x) == 0) advance_counters(adv);
    if (G.N < 2 || G.lastmask[G.N - 1] == 0) return;
    const uint32_t site = blockIdx.x * kSwapBlock + threadIdx.x;
    if (site < G.V) swap_site<kAhead>(G, site);
}

template <bool kAhead>
__global__ void __launch_bounds__(kSwapBlock)
k_swap_apply_batched(const BatchPlan plan, const Advance adv) {
    if ((blockIdx.x | threadIdx.x) == 0) advance_counters(adv);
    const BlockPlace at = locate<false>(plan, blockIdx.x);
    const GroupDev G = group_record<false>(plan, at.gi);
    if (G.N < 2 || G.lastmask[G.N - 1] == 0) return;
    const uint32_t site = at.local * kSwapBlock + threadIdx.x;
    if (site < G.V) swap_site<kAhead>(G, site);
}

// ---------------------------------------------------------------------------
// Readings: the groups' regions into one packed buffer in pinned host memory,
// so that a MiB of them costs one launch and one wait instead of one copy per
// group: energies, sums and exchange counts of 64 groups of 32 slots
// took 4.5 ms that way and take 1.  Bound by launch and bus latency, on
// megabytes by the bus.
// ---------------------------------------------------------------------------
__global__ void __launch_bounds__(256)
k_zero_meas(const GroupDev* __restrict__ groups) {
    const GroupDev G = uniform_record(groups + blockIdx.x);
    for (uint32_t i = threadIdx.x; i < G.N * kCntStride; i += 256) G.meas[i] = 0;
}

__device__ __forceinline__ void read_raw(uint64_t* __restrict__ out, const void* src, size_t words,
                                         uint32_t first, uint32_t step) {
    for (size_t i = first; i < words; i += step) out[i] = static_cast<const uint64_t*>(src)[i];
}

__global__ void __launch_bounds__(256)
k_read(const GroupDev* __restrict__ groups, Reading what, const uint64_t* __restrict__ offsets,
       uint8_t* __restrict__ out) {
    const GroupDev G = uniform_record(groups + blockIdx.x);
    uint8_t* o = out + offsets[blockIdx.x];
    const uint32_t first = blockIdx.y * 256 + threadIdx.x, step = gridDim.y * 256;
    const uint32_t N = G.N, pairs = N > 1 ? N - 1 : 1;
    const int32_t V = (int32_t)G.V;
    uint64_t* o64 = (uint64_t*)o;
    switch (what) {
        case Reading::energy:
            for (uint32_t i = first; i < N * 64; i += step) {
                const int32_t* c = G.meas + (i >> 6) * kCntStride + (i & 63u);
                ((int2*)o)[i] = make_int2(2 * V - 2 * c[0], V - 2 * c[64]);
            }
            break;
        case Reading::overlap:
            for (uint32_t i = first; i < N * 32; i += step)
                ((int64_t*)o)[i] =
                    (int64_t)V - 2 * (int64_t)G.meas[(i >> 5) * kCntStride + 128 + (i & 31u)];
            break;
        case Reading::walkers:
            for (uint32_t i = first; i < N * 64; i += step) o[i] = (uint8_t)G.walker[i];
            break;
        case Reading::accepts: read_raw(o64, G.acc, pairs, first, step); break;
        case Reading::swaplog:
            read_raw(o64, G.swaplog, (size_t)G.log_cap * pairs, first, step);
            break;
        case Reading::roundtrips:
            read_raw(o64, G.rt, (size_t)N * 64 * (sizeof(RoundTrip) / 8), first, step);
            break;
        case Reading::sums: read_raw(o64, G.sums, (size_t)N * kSumStride, first, step); break;
        case Reading::hist: read_raw(o64, G.hist, (size_t)N * kHistBins / 2, first, step); break;
    }
}

// ---------------------------------------------------------------------------
// Initialisation.
// ---------------------------------------------------------------------------
// Couplings: lane j has J_{i,d} = -1 iff bit 0 of word 0 of Philox with
// counter (i, d, 3<<24, 0) under key j_seed[j] is set (i = x + L*y;
// d = 0: +x bond, d = 1: +y bond).
__global__ void k_init_couplings(const GroupDev G) {
    const uint32_t b = blockIdx.x * blockDim.x + threadIdx.x;
    const uint32_t P = G.L * G.L;
    if (b >= 2 * P) return;
    const uint32_t d = b / P, i = b - d * P;
    uint64_t w = 0;
    for (int j = 0; j < 64; ++j) {
        const uint64_t key = G.jseed[j];
        const uint4 o = philox(make_uint4(i, d, 3u << 24, 0u), (uint32_t)key, (uint32_t)(key >> 32));
        w |= (uint64_t)(o.x & 1u) << j;
    }
    (d == 0 ? G.Jx : G.Jy)[i] = w;
}

// Spins: word(s, g) = o0 | o1<<32 of Philox with counter (s, 0, 2<<24 | g, gid).
__global__ void k_init_spins(const GroupDev G) {
    const uint32_t s = blockIdx.x * blockDim.x + threadIdx.x;
    const uint32_t g = blockIdx.y;
    if (s >= G.V) return;
    const uint4 o = philox(make_uint4(s, 0u, (2u << 24) | g, G.gid), G.key0, G.key1);
    G.spins[(size_t)g * G.V + s] = lo_hi(o.x, o.y);
}

// Walkers at their own slots, trackers, counters and sums cleared; walker 0
// starts its clock at slot 0.
__global__ void k_init_state(const GroupDev G) {
    const uint32_t j = threadIdx.x;
    const uint32_t N = G.N;
    for (uint32_t g = 0; g < N; ++g) {
        G.walker[g * 64 + j] = g;
        RoundTrip r;
        r.state = (g == 0) ? 1u : 0u;
        r.t_last = 0;
        r.count = 0;
        r.pad = 0;
        r.sum = 0;
        G.rt[g * 64 + j] = r;
        for (int k = j; k < kCntStride; k += 64) G.cnt[g * kCntStride + k] = 0;
        for (int k = j; k < kSumStride; k += 64) G.sums[(size_t)g * kSumStride + k] = 0;
        for (int k = j; k < kHistBins; k += 64) G.hist[(size_t)g * kHistBins + k] = 0;
        G.E[(g * 64 + j) * 2 + 0] = 0;
        G.E[(g * 64 + j) * 2 + 1] = 0;
    }
    const uint32_t pairs = N > 1 ? N - 1 : 1;  // the acc region has max(N-1, 1) entries
    for (uint32_t g = j; g < N; g += 64) G.lastmask[g] = 0;
    for (uint32_t g = j; g < pairs; g += 64) G.acc[g] = 0;
    const size_t nlog = (size_t)G.log_cap * (N > 1 ? N - 1 : 1);
    for (size_t i = j; i < nlog; i += 64) G.swaplog[i] = 0;
}

__global__ void k_philox(const uint32_t* in, uint32_t* out, uint32_t n) {
    const uint32_t i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const uint32_t* a = in + 6 * (size_t)i;
    const uint4 o = philox(make_uint4(a[0], a[1], a[2], a[3]), a[4], a[5]);
    uint32_t* b = out + 4 * (size_t)i;
    b[0] = o.x;
    b[1] = o.y;
    b[2] = o.z;
    b[3] = o.w;
}


// Random-number ceiling: thread i generates `blocks` Philox blocks with the
// counters the colour pass uses (a per-thread first word, block-uniform
// others: (i, 0, b, 0)) and stores the xor of all their output words.
__global__ void __launch_bounds__(256)
k_philox_probe(uint32_t* out, uint32_t n, uint32_t blocks, uint32_t k0, uint32_t k1) {
    const uint32_t i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    uint32_t x = 0;
#pragma unroll 1
    for (uint32_t b = 0; b < blocks; ++b) {
        const uint4 o = philox(make_uint4(i, 0u, b, 0u), k0, k1);
        x ^= xor3(o.x, o.y, o.z) ^ o.w;
    }
    out[i] = x;
}

}  // namespace

// ------------------------------- launchers ---------------------------------

hipError_t launch_init_couplings(const GroupDev& g, hipStream_t s) {
    const uint32_t n = 2 * g.L * g.L;
    hipLaunchKernelGGL(k_init_couplings, dim3((n + 63) / 64), dim3(64), 0, s, g);
    return hipGetLastError();
}
hipError_t launch_init_spins(const GroupDev& g, hipStream_t s) {
    hipLaunchKernelGGL(k_init_spins, dim3((g.V + 255) / 256, g.N), dim3(256), 0, s, g);
    return hipGetLastError();
}
hipError_t launch_init_state(const GroupDev& g, hipStream_t s) {
    hipLaunchKernelGGL(k_init_state, dim3(1), dim3(64), 0, s, g);
    return hipGetLastError();
}
hipError_t launch_half_sweep(const GroupDev& g, uint32_t colour, const uint32_t* ctr,
                             uint32_t t_add, hipStream_t s) {
    hipLaunchKernelGGL(k_half_sweep, dim3(sweep_blocks_per_slot(g.V, g.tile), g.N), dim3(kSweepBlock), 0, s,
                       g, colour, ctr, t_add);
    return hipGetLastError();
}
hipError_t launch_energy(const GroupDev& g, int32_t* cnt, hipStream_t s) {
    const EnergyWalks w = energy_walks(g.L * g.L, g.Ltau, (uint64_t)g.N * g.V);
    const dim3 grid(energy_blocks_per_slot(g.L * g.L, w.tiles), g.N), block(kEnergyBlock);
    if (w.planes <= (uint32_t)kEnergyShort)
        hipLaunchKernelGGL(k_energy<kEnergyShort>, grid, block, 0, s, g, cnt, w);
    else
        hipLaunchKernelGGL(k_energy<kEnergyLong>, grid, block, 0, s, g, cnt, w);
    return hipGetLastError();
}
hipError_t launch_pt(const GroupDev& g, const uint32_t* ctr, hipStream_t s) {
    hipLaunchKernelGGL(k_pt, dim3(1), dim3(kPtBlock), 0, s, g, ctr);
    return hipGetLastError();
}
hipError_t launch_swap_apply(const GroupDev& g, const Advance& adv, hipStream_t s) {
    const uint32_t blocks = swap_blocks(g.V);
    if (blocks <= kSwapAheadBlocks)
        hipLaunchKernelGGL(k_swap_apply<true>, dim3(blocks), dim3(kSwapBlock), 0, s, g, adv);
    else
        hipLaunchKernelGGL(k_swap_apply<false>, dim3(blocks), dim3(kSwapBlock), 0, s, g, adv);
    return hipGetLastError();
}
hipError_t launch_zero_meas(const GroupDev* groups, uint32_t n_groups, hipStream_t s) {
    hipLaunchKernelGGL(k_zero_meas, dim3(n_groups), dim3(256), 0, s, groups);
    return hipGetLastError();
}
hipError_t launch_read(const GroupDev* groups, uint32_t n_groups, Reading what,
                       const uint64_t* offsets, void* out, hipStream_t s) {
    constexpr uint32_t kSplit = 8;  // blocks per group
    hipLaunchKernelGGL(k_read, dim3(n_groups, kSplit), dim3(256), 0, s, groups, what, offsets,
                       (uint8_t*)out);
    return hipGetLastError();
}
hipError_t launch_philox(const uint32_t* in, uint32_t* out, uint32_t n, hipStream_t s) {
    if (n == 0) return hipSuccess;
    hipLaunchKernelGGL(k_philox, dim3((n + 63) / 64), dim3(64), 0, s, in, out, n);
    return hipGetLastError();
}
hipError_t launch_philox_probe(uint32_t* out, uint32_t n, uint32_t blocks, uint64_t key,
                              hipStream_t s) {
    if (n == 0) return hipSuccess;
    hipLaunchKernelGGL(k_philox_probe, dim3((n + 255) / 256), dim3(256), 0, s, out, n, blocks,
                       (uint32_t)key, (uint32_t)(key >> 32));
    return hipGetLastError();
}
hipError_t launch_half_sweep_batched(const BatchPlan& plan, uint32_t colour, const uint32_t* ctr,
                                     uint32_t t_add, hipStream_t s) {
    if (plan.n_blocks == 0) return hipSuccess;
    if (plan.same_shape)
        hipLaunchKernelGGL(k_half_sweep_batched<true>, dim3(plan.n_blocks), dim3(kSweepBlock), 0, s,
                           plan, colour, ctr, t_add);
    else
        hipLaunchKernelGGL(k_half_sweep_batched<false>, dim3(plan.n_blocks), dim3(kSweepBlock), 0,
                           s, plan, colour, ctr, t_add);
    return hipGetLastError();
}
hipError_t launch_chunk_fused(const BatchPlan& slots, const uint32_t* ctr, uint32_t n_sweeps,
                              const FusedShape& f, hipStream_t s) {
    if (slots.n_blocks == 0) return hipSuccess;
    const size_t lds = (size_t)f.lds_words * sizeof(uint64_t);
    if (lds) {
        if (lds > 48 * 1024) {
            // always the most that any context needs: the limit belongs to the
            // kernel, and another thread's context may be about to launch
            hipError_t e = hipFuncSetAttribute((const void*)k_chunk_fused<true>,
                                               hipFuncAttributeMaxDynamicSharedMemorySize,
                                               (int)(kFusedLdsWords * sizeof(uint64_t)));
            if (e != hipSuccess) return e;
        }
        hipLaunchKernelGGL(k_chunk_fused<true>, dim3(slots.n_blocks), dim3(f.threads), lds, s,
                           slots, ctr, n_sweeps);
    } else {
        hipLaunchKernelGGL(k_chunk_fused<false>, dim3(slots.n_blocks), dim3(f.threads), 0, s, slots,
                           ctr, n_sweeps);
    }
    return hipGetLastError();
}

hipError_t launch_energy_batched(const BatchPlan& plan, uint32_t eplanes, bool reading,
                                 hipStream_t s) {
    if (plan.n_blocks == 0) return hipSuccess;
    if (eplanes <= (uint32_t)kEnergyShort)
        hipLaunchKernelGGL(k_energy_batched<kEnergyShort>, dim3(plan.n_blocks), dim3(kEnergyBlock),
                           0, s, plan, (uint32_t)reading);
    else
        hipLaunchKernelGGL(k_energy_batched<kEnergyLong>, dim3(plan.n_blocks), dim3(kEnergyBlock),
                           0, s, plan, (uint32_t)reading);
    return hipGetLastError();
}
hipError_t launch_pt_batched(const GroupDev* groups, uint32_t n_groups, const uint32_t* ctr,
                             hipStream_t s) {
    if (n_groups == 0) return hipSuccess;
    hipLaunchKernelGGL(k_pt_batched, dim3(n_groups), dim3(kPtBlock), 0, s, groups, ctr);
    return hipGetLastError();
}
hipError_t launch_advance(const Advance& adv, hipStream_t s) {
    hipLaunchKernelGGL(k_advance, dim3(1), dim3(64), 0, s, adv);
    return hipGetLastError();
}
hipError_t launch_swap_apply_batched(const BatchPlan& plan, const Advance& adv, hipStream_t s) {
    if (plan.n_blocks == 0) return launch_advance(adv, s);  // groups of one slot only
    if (plan.n_blocks <= kSwapAheadBlocks)
        hipLaunchKernelGGL(k_swap_apply_batched<true>, dim3(plan.n_blocks), dim3(kSwapBlock), 0, s,
                           plan, adv);
    else
        hipLaunchKernelGGL(k_swap_apply_batched<false>, dim3(plan.n_blocks), dim3(kSwapBlock), 0, s,
                           plan, adv);
    return hipGetLastError();
}

}  // namespace qsg
