// Level entries of the ladders the host builds: every one is the start of a
// handler, that of the level's truth table over the class codes; and before
// every ladder is set no sweep is launched.
#include "host_runtime.h"

#include <cmath>
#include <cstdio>
#include <vector>

namespace qsg {
std::vector<GroupDev> made;
int sweeps = 0;
hipError_t launch_init_couplings(const GroupDev&, hipStream_t) { return host::launched(); }
hipError_t launch_init_spins(const GroupDev&, hipStream_t) { return host::launched(); }
hipError_t launch_init_state(const GroupDev& g, hipStream_t) {
    made.push_back(g);
    return host::launched();
}
hipError_t launch_half_sweep(const GroupDev&, uint32_t, const uint32_t*, uint32_t, hipStream_t) {
    ++sweeps;
    return host::launched();
}
hipError_t launch_advance(const Advance&, hipStream_t) { return host::launched(); }
}  // namespace qsg

// class code of (n_s, n_t) in a regime, or -1 (accepted outright)
int code(uint32_t regime, int ns, int nt) {
    if (regime == 0) return nt == 0 ? ns : nt == 1 && ns < 2 ? 5 + ns : -1;
    if (regime == 1) return nt == 0 ? (ns < 4 ? ns : -1) : nt == 1 ? (ns < 2 ? 4 + ns : -1) : ns < 1 ? 6 : -1;
    return nt == 0 ? (ns < 3 ? 4 + ns : -1) : ns < 2 ? (nt == 1 ? ns : 2 + ns) : -1;
}

int main() {
    constexpr uint32_t N = 2;
    std::vector<qsg_group_desc> d(3);
    for (uint32_t i = 0; i < 3; ++i) {
        d[i] = qsg_group_desc{};
        d[i].L = 4;
        d[i].L_tau = 8;
        d[i].beta = i == 1 ? 1e-3 : 4.0;
        d[i].n_gamma = N;
        d[i].swap_table_cap = 1;
        d[i].ladder_kind = i == 2 ? QSG_LADDER_K : QSG_LADDER_GAMMA;
    }
    qsg_run_config cfg{};
    cfg.swaplog_cap = 1;
    // one value to a ladder: exchange tables of equal slots are empty
    const size_t bytes = qsg_workspace_bytes(d.data(), 3, &cfg);
    void* ws = std::aligned_alloc(256, (bytes + 255) / 256 * 256);
    std::memset(ws, 0, bytes);
    qsg_ctx* c = nullptr;
    if (qsg_create(d.data(), 3, &cfg, ws, bytes, nullptr, &c) || qsg_init_spins(c)) return 1;
    int slots = 0, regimes = 0;
    for (int trial = 0; trial < 200; ++trial) {
        for (uint32_t i = 0; i < 3; ++i) {
            // time couplings from frozen to vanishing, spaces likewise
            const double value = std::exp(-14.0 + 20.0 * trial / 199.0 + 0.01 * i);
            const std::vector<double> lad(N, value);
            if (i == 2 ? qsg_set_k_ladder(c, i, lad.data()) : qsg_set_gamma_ladder(c, i, lad.data()))
                return 2;
            if (trial == 0 && i < 2 && (qsg_sweep(c, 1, QSG_PLAIN) != QSG_E_STATE || qsg::sweeps)) {
                std::printf("a sweep ran before every ladder was set\n");
                return 3;
            }
            for (uint32_t g = 0; g < N; ++g, ++slots) {
                const uint32_t* t = qsg::made[i].thr + g * qsg::kThrStride;
                const uint32_t regime = t[15];
                if (regime > 2) return 4;
                regimes |= 1 << regime;
                for (int level = 0; level < 32; ++level) {
                    const uint32_t e = t[qsg::kLevelEntries + level / 2] >> 16 * (level % 2) & 0xFFFF;
                    const uint32_t table = (e - qsg::kHandlerSkip) / qsg::kHandlerBytes;
                    if (e < qsg::kHandlerSkip || (e - qsg::kHandlerSkip) % qsg::kHandlerBytes ||
                        table > 127 || (e & qsg::kEntryMask) != e) {
                        std::printf("entry %u\n", e);
                        return 5;
                    }
                    for (int k = 0; k < 15; ++k) {
                        const int cls = code(regime, k / 3, k % 3);
                        if (cls < 0 ? t[k] != 0xFFFFFFFFu
                                    : (table >> cls & 1) != (t[k] >> (31 - level) & 1))
                            return 6;
                    }
                }
            }
        }
    }
    if (qsg_sweep(c, 1, QSG_PLAIN) || !qsg::sweeps) return 7;
    std::printf("%d slots, regimes %d\n", slots, regimes);
    return regimes == 7 ? 0 : 8;
}
