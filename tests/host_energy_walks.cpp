// Depth of the energy pass's walks: tiles cover L_tau, no slot's waves crowd
// its counters while deeper walks are there, and whole 64-plane walks from 6.5
// M words on.
#include <cstdio>

#include "host_runtime.h"

int main() {
    using namespace qsg;
    for (uint32_t L = 2; L <= 256; L += L < 32 ? 2 : 32)
        for (uint32_t Lt : {2u, 4u, 6u, 16u, 34u, 64u, 90u, 94u, 128u, 190u, 256u, 2046u, 2048u, 65536u})
            for (uint64_t slots : {1ull, 3ull, 40ull, 3000ull}) {
                const uint64_t words = slots * L * L * Lt;
                const EnergyWalks w = energy_walks(L * L, Lt, words);
                const uint64_t waves = (uint64_t)L * L * w.tiles / 64;
                const char* what = nullptr;
                if (w.tiles == 0 || w.tiles * w.planes - w.n_short != Lt || w.n_short >= w.tiles ||
                    w.planes > (uint32_t)kEnergyLong || (w.n_short && w.planes < 3))
                    what = "tiles do not cover the slot";
                if (waves > 256 && w.tiles > (Lt + 63) / 64) what = "waves crowd a slot";
                if (words >= 6500000 && Lt % 64 == 0 && w.planes != 64) what = "not 64 planes";
                if (what) {
                    std::printf("L %u L_tau %u slots %llu: %s (%u tiles of %u)\n", L, Lt,
                                (unsigned long long)slots, what, w.tiles, w.planes);
                    return 1;
                }
            }
    return 0;
}
