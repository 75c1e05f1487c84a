// Internal layout shared by the host API and the HIP kernels.
#pragma once

#include <hip/hip_runtime.h>

#include <cstddef>
#include <cstdint>

namespace qsg {

// Per-(walker, lane) round-trip tracker; same layout as qsg_roundtrip.
struct RoundTrip {
    uint32_t state;
    uint32_t t_last;
    uint32_t count;
    uint32_t pad;
    uint64_t sum;
};

// Counters the energy pass accumulates per slot: unsatisfied space bonds and
// time bonds per lane, differing lane pairs per pair.
constexpr int kCntStride = 64 + 64 + 32;  // int32 per slot
// Per-slot measurement sums: Bsp[64], Bt[64], q[32], q^2[32] as int64.
constexpr int kSumStride = 192;
// Per-slot table: [0, 15) thresholds of the fifteen classes, [15] the class
// regime, [16, 32) the handler entries of the 32 comparison levels, most
// significant first, two 16-bit entries to a word (the word of Philox block
// q).  A level's truth table (7 bits) has bit c set when the threshold of
// class code c has a 1 at that level; table i's handler starts kHandlerSkip +
// i * kHandlerBytes after the address the colour pass jumps from.
constexpr int kThrStride = 32;
constexpr int kLevelEntries = 16;
constexpr uint32_t kHandlerBytes = 32;
constexpr uint32_t kHandlerSkip = 12;
constexpr uint32_t kEntryMask = 127 * kHandlerBytes | kHandlerSkip;
constexpr uint32_t level_entry(uint32_t table) { return kHandlerSkip + table * kHandlerBytes; }
// Histogram of the unsatisfied time bonds u = (V - Bt)/2 per slot, taken at
// every PT step before the exchanges: bin = u * kHistBins / (V + 1).
constexpr int kHistBins = 1024;

// Exact division by a fixed d for x < 2^31: q = mulhi(x, m) >> s, or
// x >> s when m == 0 (d a power of two).
struct Divisor {
    uint32_t m, s;
};

inline Divisor make_divisor(uint32_t d) {
    Divisor r{0, 0};
    uint32_t a = 0;
    while ((1ull << (a + 1)) <= d) ++a;  // a = floor(log2 d)
    if ((1u << a) == d) {
        r.s = a;
    } else {
        // d in (2^a, 2^(a+1)): m = ceil(2^(32+a)/d) < 2^32, exact for x < 2^31
        r.m = (uint32_t)(((1ull << (32 + a)) + d - 1) / d);
        r.s = a;
    }
    return r;
}

// Column walks of the energy pass: Ltau planes in `tiles` tau tiles of
// `planes` planes, the first `n_short` of them one plane less.
struct EnergyWalks {
    uint32_t tiles, planes, n_short;
};

// Everything a kernel needs to know about one group.  Lives on the host
// (plain launches pass it by value) and in a device array (batched
// launches index it).
struct GroupDev {
    uint32_t L, Ltau, N, gid;
    uint32_t key0, key1;  // Monte Carlo key (mc_seed lo, hi)
    uint32_t V;           // words per slot = L*L*Ltau
    uint32_t sw_cap;      // entries per exchange table
    uint32_t log_cap;     // rows of the swap log
    uint32_t q_split;     // colour-pass schedule: Philox blocks before packing
    uint32_t tile;        // colour-pass schedule: tau planes per column walk (even, divides Ltau)
    uint32_t exch_all;    // PT energy: 0 time bonds (Gamma ladder), 1 all bonds (k ladder)
    uint32_t anti;        // 1: antiperiodic along tau (the wrapping time bond flips sign)
    EnergyWalks ewalk;    // energy pass, batched
    Divisor div_half_plane, div_half_row, div_plane, div_row;
    Divisor div_blocks;   // colour-pass blocks per slot (sweep_blocks_per_slot(V, tile))
    uint64_t* spins;          // [N][Ltau][L][L]
    uint64_t* Jx;             // [L*L]
    uint64_t* Jy;             // [L*L]
    const uint64_t* jseed;    // [64] coupling keys
    uint32_t* thr;            // [N][kThrStride] thresholds, regime, handler entries
    uint32_t* sw_thr;         // [N-1][sw_cap]
    uint32_t* sw_len;         // [N-1]
    uint32_t* sw_eq;          // [N-1]
    int32_t* cnt;             // [N][kCntStride]
    int32_t* E;               // [N][64][2] current (Bsp, Bt)
    uint32_t* walker;         // [N][64]
    RoundTrip* rt;            // [N walkers][64 lanes]
    uint64_t* acc;            // [N-1]
    uint64_t* swaplog;        // [log_cap][N-1]
    int64_t* sums;            // [N][kSumStride]
    uint64_t* lastmask;       // [N] masks of the latest PT step (+ any flag at [N-1])
    int32_t* meas;            // [N][kCntStride] scratch for on-demand measurement
    uint32_t* hist;           // [N][kHistBins]
};

// Launchers (qsg_kernels.hip).  All enqueue on `s` and return the launch
// status.  `ctr` is the device pair (sweeps done, PT steps done); sweep and
// PT kernels use ctr[0] + t_add and ctr[1] as their indices.
hipError_t launch_init_couplings(const GroupDev& g, hipStream_t s);
hipError_t launch_init_spins(const GroupDev& g, hipStream_t s);
hipError_t launch_init_state(const GroupDev& g, hipStream_t s);
// The colour pass follows the group's schedule G.q_split: Philox blocks every
// word goes through before the words still undecided are packed into the
// first waves of the block (16: no packing; the fused chunk never packs).
// Results do not depend on it.
hipError_t launch_half_sweep(const GroupDev& g, uint32_t colour, const uint32_t* ctr,
                             uint32_t t_add, hipStream_t s);
hipError_t launch_energy(const GroupDev& g, int32_t* cnt, hipStream_t s);
hipError_t launch_pt(const GroupDev& g, const uint32_t* ctr, hipStream_t s);
// The device counters (sweeps done, PT steps done) and what to add to them.
struct Advance {
    uint32_t* ctr;
    uint32_t dt, dp;
};
hipError_t launch_advance(const Advance& adv, hipStream_t s);
// The exchange pass is the last launch of a PT step and advances the counters
// (adv.ctr null: the launch for another group does).
hipError_t launch_swap_apply(const GroupDev& g, const Advance& adv, hipStream_t s);

hipError_t launch_philox(const uint32_t* in, uint32_t* out, uint32_t n, hipStream_t s);
hipError_t launch_philox_probe(uint32_t* out, uint32_t n, uint32_t blocks, uint64_t key,
                              hipStream_t s);

// Batched: one launch per pass over all groups.  `prefix[i]` is the first
// block of group i (prefix[n_groups] = total blocks).
// Group of a block and the block's index within the group.
struct BlockEntry {
    uint32_t gi, local;
};

struct BatchPlan {
    const GroupDev* groups;  // device array [n_groups]
    const uint32_t* prefix;  // device array [n_groups + 1]
    // optional device array [n_blocks]: every block's group and index in
    // it, so that a block of an ensemble of unequal groups finds its group
    // with one load instead of a search of `prefix`
    const BlockEntry* block_map;
    uint32_t n_groups;
    uint32_t n_blocks;
    // per_group > 0 when every group has exactly per_group blocks: a block
    // then finds its group by one scalar division (span divides by
    // per_group) instead of a search of `prefix`
    uint32_t per_group;
    Divisor span;
    // same_shape != 0 when every group's record equals `first` up to its
    // Philox identity (gid, key0, key1) and pointers that advance by
    // `stride` bytes from one group to the next: a block then builds its
    // record from this kernel argument instead of loading it first
    uint32_t same_shape;
    uint64_t stride;
    GroupDev first;
};

// Record i with its pointers moved back by `shift` bytes and its Philox
// identity cleared: equal for all groups of one shape (shift = i * stride).
inline bool same_but_identity(const GroupDev& a, const GroupDev& b, uint64_t shift) {
    auto ptr = [shift](const void* p, const void* q) {
        return (uint64_t)(uintptr_t)p == (uint64_t)(uintptr_t)q + shift;
    };
    auto div = [](Divisor x, Divisor y) { return x.m == y.m && x.s == y.s; };
    return a.L == b.L && a.Ltau == b.Ltau && a.N == b.N && a.V == b.V && a.sw_cap == b.sw_cap &&
           a.log_cap == b.log_cap && a.q_split == b.q_split && a.tile == b.tile &&
           a.exch_all == b.exch_all && a.ewalk.tiles == b.ewalk.tiles &&
           a.anti == b.anti && div(a.div_half_plane, b.div_half_plane) &&
           div(a.div_half_row, b.div_half_row) && div(a.div_plane, b.div_plane) &&
           div(a.div_row, b.div_row) && div(a.div_blocks, b.div_blocks) &&
           ptr(a.spins, b.spins) && ptr(a.Jx, b.Jx) && ptr(a.Jy, b.Jy) && ptr(a.jseed, b.jseed) &&
           ptr(a.thr, b.thr) && ptr(a.sw_thr, b.sw_thr) && ptr(a.sw_len, b.sw_len) &&
           ptr(a.sw_eq, b.sw_eq) && ptr(a.cnt, b.cnt) && ptr(a.E, b.E) &&
           ptr(a.walker, b.walker) && ptr(a.rt, b.rt) && ptr(a.acc, b.acc) &&
           ptr(a.swaplog, b.swaplog) && ptr(a.sums, b.sums) && ptr(a.lastmask, b.lastmask) &&
           ptr(a.meas, b.meas) && ptr(a.hist, b.hist);
}

// Set the plan's shared-shape fields from the host copy of the records
// (again whenever a record changes).
inline void set_plan_shape(BatchPlan& p, const GroupDev* records, uint32_t n_groups) {
    p.same_shape = 0;
    p.stride = 0;
    p.first = GroupDev{};
    if (n_groups == 0) return;
    const uint64_t base = (uint64_t)(uintptr_t)records[0].spins;
    const uint64_t stride = n_groups > 1 ? (uint64_t)(uintptr_t)records[1].spins - base : 0;
    for (uint32_t i = 0; i < n_groups; ++i)
        if (!same_but_identity(records[i], records[0], (uint64_t)i * stride)) return;
    p.same_shape = 1;
    p.stride = stride;
    p.first = records[0];
}

// The plan of a batched launch from the host copy of its prefix sums and
// of the group records.
inline BatchPlan make_plan(const GroupDev* groups, const uint32_t* d_prefix,
                           const uint32_t* prefix, uint32_t n_groups, const GroupDev* records) {
    BatchPlan p{};
    p.groups = groups;
    p.prefix = d_prefix;
    p.n_groups = n_groups;
    p.n_blocks = prefix[n_groups];
    const uint32_t first = n_groups ? prefix[1] - prefix[0] : 0;
    bool equal = first > 0;
    for (uint32_t i = 1; equal && i < n_groups; ++i) equal = prefix[i + 1] - prefix[i] == first;
    if (equal) {
        p.per_group = first;
        p.span = make_divisor(first);
    }
    set_plan_shape(p, records, n_groups);
    return p;
}
hipError_t launch_half_sweep_batched(const BatchPlan& plan, uint32_t colour, const uint32_t* ctr,
                                     uint32_t t_add, hipStream_t s);
// eplanes: the deepest walk among the plan's groups.  The counts are added
// to the groups' pass counters, or (`reading`) to their `meas` arrays.
hipError_t launch_energy_batched(const BatchPlan& plan, uint32_t eplanes, bool reading,
                                 hipStream_t s);
hipError_t launch_zero_meas(const GroupDev* groups, uint32_t n_groups, hipStream_t s);
// Readings of groups[0 .. n_groups) into one buffer that device and host see:
// group i's starts at byte offsets[i], in the C ABI's layout.
enum class Reading : uint32_t { energy, overlap, walkers, accepts, swaplog, roundtrips, sums, hist };
hipError_t launch_read(const GroupDev* groups, uint32_t n_groups, Reading what,
                       const uint64_t* offsets, void* out, hipStream_t s);
// Fused sweeps over every slot (one block per slot, `slots.prefix` counts
// slots per group): n_sweeps sweeps in one launch.
constexpr uint32_t kFusedBlock = 1024;
constexpr uint32_t kFusedLdsWords = 20000;  // 156 KiB of a CU's 160
struct FusedShape {
    uint32_t threads;    // per block, whole waves
    uint32_t lds_words;  // spins and couplings of the largest slot; 0: run from global memory
};
// max_v: words of the largest slot; max_lds: its words and couplings, V + 2
// L^2.  As few rounds of words as 1024 threads allow, with as few threads as
// these rounds need.
inline FusedShape fused_shape(uint32_t max_v, uint32_t max_lds) {
    const uint32_t half = max_v / 2, rounds = (half + kFusedBlock - 1) / kFusedBlock;
    const uint32_t threads = ((half + rounds - 1) / rounds + 63) / 64 * 64;
    return {threads, max_lds <= kFusedLdsWords ? max_lds : 0};
}
// A chunk graph holds the fused launch instead of the colour passes if no
// slot has more words than this.  A colour pass of a graph lasts at least 5.7
// us, a fused one 1.1 us and 2.3 per 1024 words on the one CU that a slot is
// on: they meet at about 3000 words a slot where slots are few, later where
// they are many.  100 sweeps, passes / fused: 1.38 / 0.99 ms for 16 slots of
// 2048 words, 1.96 / 1.14 for 256, 4.42 / 2.86 for 1024; 3.42 / 2.67 for 600
// of 2160; but 1.41 / 1.74 for 16 of 4096.
constexpr uint32_t kFusedGraphWords = 2560;
hipError_t launch_chunk_fused(const BatchPlan& slots, const uint32_t* ctr, uint32_t n_sweeps,
                              const FusedShape& shape, hipStream_t s);
// Column-walk depth of the colour pass (tau planes per thread; each thread
// updates tile/2 words): the largest allowed, and the default for a launch
// over `words` words.  Deep walks save loads and index work per word, shallow
// ones give more waves, and a launch of few waves lasts as long as one thread
// takes: the default is the deepest of 8, 4, 2 that leaves two rounds of
// waves for the chip (2 x 8192).  Measured per pass at depths 8 / 4 / 2: 14.1
// / 8.5 / 5.8 us on 33 k words, 17.3 / 12.6 / 12.1 on 1 M, 21.7 / 20.0 / 19.5
// on 2 M, 33.5 / 30.6 / 31.9 on 4 M, 52.7 / 52.6 / 56.9 on 8 M, 93 / 97 / 107
// on 17 M.
constexpr uint32_t kMaxTile = 32;
inline uint32_t default_tile(uint64_t words) {
    constexpr uint64_t kWaves = 2 * 8192, kLanes = 64;
    uint32_t tile = 8;
    while (tile > 2 && words < kWaves * kLanes * tile) tile /= 2;
    return tile;
}
// Largest power of two <= cap that divides Ltau (Ltau is even: at least 2).
inline uint32_t tile_for(uint32_t Ltau, uint32_t cap) {
    uint32_t t = 2;
    while (t * 2 <= cap && Ltau % (t * 2) == 0) t *= 2;
    return t;
}
// Energy pass: each thread walks one column through one tau tile of at most
// kEnergyLong planes; walks of at most kEnergyShort planes run in an
// instantiation with fewer counter planes.
constexpr int kEnergyShort = 16;
constexpr int kEnergyLong = 64;
constexpr int kEnergyBlock = 256;
inline EnergyWalks walks_of_depth(uint32_t Ltau, uint32_t depth) {
    EnergyWalks w;
    w.tiles = (Ltau + depth - 1) / depth;
    w.planes = (Ltau + w.tiles - 1) / w.tiles;
    w.n_short = w.tiles * w.planes - Ltau;
    return w;
}
// The loads of the next batch of four planes run ahead only on walks of whole
// pairs of batches.
__host__ __device__ inline bool walks_ahead(const EnergyWalks& w) {
    return w.planes % 8 == 0 && w.n_short == 0;
}
// Depth of the walks of a launch over `words` words in slots of P columns:
// every wave ends with transposes that cost as much as 16 planes, so the
// deepest that leaves the chip enough waves.  Tiles need not divide Ltau
// (their sizes differ by one plane): where they had to, 3 M words at Ltau = 90
// (walks of 2 planes) took 75 us instead of 15.  Measured after exchange
// passes, at depths 4 / 8 / 16 / 32 / 64 (us): 6.3 / 6.7 / 7.4 / 11 / 12 on 33 k
// words, 8.0 / 7.3 / 8.8 / 13 / 16 on 324 k, 14 / 9.2 / 8.6 / 11 / 16 on 1 M, 21 /
// 13 / 10 / 11 / 16 on 2 M, 46 / 28 / 22 / 20 / 24 on 5 M, 510 / 278 / 200 / 183 /
// 182 on 67 M and 360 / 291 / 257 (depths 16 / 32 / 64) on 113 M.  Two things
// ask for deeper walks:
// - All waves of a slot add to the same 160 counters, one after the other: 94 /
//   50 / 29 / 21 / 19 us on one slot of 1.2 M words, whose waves number 4608 at
//   depth 4 and 288 at 64; 81 / 44 / 22 / 18 / 17 on six slots of 0.5 M.
// - From 6.5 M words on, 64 planes read ahead beat 32: 22.8 / 21.8 us (depths 32
//   / 64) on 6.6 M, 31 / 28 on 13 M, 61 / 50 on 25 M; not so where the walks
//   are ragged (30 / 38 on 7.8 M at Ltau = 94).
inline EnergyWalks energy_walks(uint32_t P, uint32_t Ltau, uint64_t words) {
    uint32_t depth = words >= (1ull << 26)   ? kEnergyLong
                     : words >= (1ull << 22) ? 32
                     : words >= 750000       ? 16
                     : words >= (1ull << 18) ? 8
                                             : 4;
    const uint32_t slot_waves = words >= (1ull << 21) ? 128 : 256;
    while (depth < (uint32_t)kEnergyLong && P * walks_of_depth(Ltau, depth).tiles > 64 * slot_waves)
        depth *= 2;
    if (words >= 6500000 && walks_ahead(walks_of_depth(Ltau, kEnergyLong))) depth = kEnergyLong;
    return walks_of_depth(Ltau, depth);
}
hipError_t launch_pt_batched(const GroupDev* groups, uint32_t n_groups, const uint32_t* ctr,
                             hipStream_t s);
hipError_t launch_swap_apply_batched(const BatchPlan& plan, const Advance& adv, hipStream_t s);

// Blocks one group needs in each pass (host and device agree on these).
// The colour pass gives each thread one column (x, y) of one tau tile of
// `tile` planes: V / tile threads per slot.
__host__ __device__ inline uint32_t sweep_blocks_per_slot(uint32_t V, uint32_t tile);
__host__ __device__ inline uint32_t energy_blocks_per_slot(uint32_t P, uint32_t tiles);
__host__ __device__ inline uint32_t swap_blocks(uint32_t V);

constexpr uint32_t kMaxSlots = 64;  // slots per group (the C ABI's QSG_MAX_GAMMA)
constexpr int kSweepBlock = 256;   // threads per block of a colour pass
constexpr uint32_t kWaveSize = 64;
constexpr int kPtBlock = 1024;   // one block per group: 16 waves share its slots
constexpr int kSwapBlock = 256;

}  // namespace qsg

namespace qsg {
__host__ __device__ inline uint32_t sweep_blocks_per_slot(uint32_t V, uint32_t tile) {
    return (V / tile + kSweepBlock - 1) / kSweepBlock;
}
// One thread per column (P = L^2 of them) and tau tile.
__host__ __device__ inline uint32_t energy_blocks_per_slot(uint32_t P, uint32_t tiles) {
    return (P * tiles + kEnergyBlock - 1) / kEnergyBlock;
}
__host__ __device__ inline uint32_t swap_blocks(uint32_t V) {
    return (V + kSwapBlock - 1) / kSwapBlock;
}
}  // namespace qsg
