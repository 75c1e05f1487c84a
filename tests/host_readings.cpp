// Readings with and without pinned memory: equal, and the context goes on.
#include "host_runtime.h"

#include <cstdio>
#include <vector>

namespace qsg {
// "device" state that a reading can be told by: every array holds a count of
// its own, offset by the group
template <class T>
void number(T* p, size_t n, uint64_t first) {
    for (size_t i = 0; i < n; ++i) p[i] = (T)(first + i);
}
hipError_t launch_init_couplings(const GroupDev&, hipStream_t) { return host::launched(); }
hipError_t launch_init_spins(const GroupDev&, hipStream_t) { return host::launched(); }
hipError_t launch_init_state(const GroupDev& g, hipStream_t) {
    const uint64_t id = 1000 * g.gid;
    const size_t N = g.N, pairs = N > 1 ? N - 1 : 1;
    number(g.acc, pairs, id + 1);
    number(g.swaplog, pairs * g.log_cap, id + 2);
    number(g.walker, N * 64, 3);
    number(reinterpret_cast<uint64_t*>(g.rt), N * 64 * sizeof(RoundTrip) / 8, id + 4);
    number(g.sums, N * kSumStride, id + 5);
    number(g.hist, N * kHistBins, id + 6);
    return host::launched();
}
hipError_t launch_zero_meas(const GroupDev*, uint32_t, hipStream_t) { return host::launched(); }
hipError_t launch_energy_batched(const BatchPlan& p, uint32_t, bool reading, hipStream_t) {
    for (uint32_t i = 0; reading && i < p.n_groups; ++i)
        number(p.groups[i].meas, p.groups[i].N * kCntStride, 7 * i);
    return host::launched();
}
hipError_t launch_read(const GroupDev* groups, uint32_t n, Reading what, const uint64_t* offsets,
                       void* out, hipStream_t) {
    for (uint32_t i = 0; i < n; ++i) {
        const GroupDev& g = groups[i];
        uint8_t* o = static_cast<uint8_t*>(out) + offsets[i];
        const size_t N = g.N, pairs = N > 1 ? N - 1 : 1;
        const int64_t V = g.V;
        switch (what) {
            case Reading::energy:
                for (size_t k = 0; k < N * 64; ++k) {
                    const int32_t* c = g.meas + k / 64 * kCntStride + k % 64;
                    reinterpret_cast<int32_t*>(o)[2 * k] = (int32_t)(2 * V - 2 * c[0]);
                    reinterpret_cast<int32_t*>(o)[2 * k + 1] = (int32_t)(V - 2 * c[64]);
                }
                break;
            case Reading::overlap:
                for (size_t k = 0; k < N * 32; ++k)
                    reinterpret_cast<int64_t*>(o)[k] =
                        V - 2 * (int64_t)g.meas[k / 32 * kCntStride + 128 + k % 32];
                break;
            case Reading::walkers:
                for (size_t k = 0; k < N * 64; ++k) o[k] = (uint8_t)g.walker[k];
                break;
            case Reading::accepts: std::memcpy(o, g.acc, pairs * 8); break;
            case Reading::swaplog: std::memcpy(o, g.swaplog, pairs * g.log_cap * 8); break;
            case Reading::roundtrips: std::memcpy(o, g.rt, N * 64 * sizeof(RoundTrip)); break;
            case Reading::sums: std::memcpy(o, g.sums, N * kSumStride * 8); break;
            case Reading::hist: std::memcpy(o, g.hist, N * kHistBins * 4); break;
        }
    }
    return host::launched();
}
}  // namespace qsg

int main() {
    // readings of 3, 1 and 40 slots; the last one's swap log is copied alone
    std::vector<qsg_group_desc> d(3);
    const uint32_t slots[3] = {3, 1, 40};
    for (uint32_t i = 0; i < 3; ++i) {
        d[i] = qsg_group_desc{};
        d[i].L = 4;
        d[i].L_tau = 4 + 2 * i;
        d[i].beta = 1.0;
        d[i].n_gamma = slots[i];
        d[i].group_id = i;
    }
    qsg_run_config cfg{};
    cfg.pt_every = 10;
    cfg.swaplog_cap = 2000;
    const size_t bytes = qsg_workspace_bytes(d.data(), 3, &cfg);
    void* ws = std::aligned_alloc(256, (bytes + 255) / 256 * 256);
    std::memset(ws, 0, bytes);
    std::vector<std::vector<uint8_t>> got[2];
    for (int fails = 0; fails < 2; ++fails) {
        qsg_ctx* c = nullptr;
        if (qsg_create(d.data(), 3, &cfg, ws, bytes, nullptr, &c)) return 1;
        if (qsg_init_spins(c)) return 2;
        host::fail_pinned = fails;
        for (uint32_t what = QSG_M_ENERGY; what <= QSG_M_HIST; ++what) {
            std::vector<uint8_t> out(1 << 22, 0xA5);
            const qsg_status st = qsg_measure(c, what, out.data(), out.size());
            if (st) {
                std::printf("reading %u, pinned memory %s: status %d (%s)\n", what,
                            fails ? "refused" : "there", st, qsg_last_error(c));
                return 3;
            }
            got[fails].push_back(out);
        }
        host::fail_pinned = false;
        if (qsg_init_spins(c)) return 4;  // the context is whole
        qsg_destroy(c);
    }
    for (size_t k = 0; k < got[0].size(); ++k)
        if (got[0][k] != got[1][k]) {
            std::printf("reading %zu differs\n", k + 1);
            return 5;
        }
    std::printf("%d pinned allocations, %d frees\n", host::pinned_allocs, host::pinned_frees);
    return 0;
}
