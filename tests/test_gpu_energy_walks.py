"""Bond sums and overlaps of the energy pass at every walk depth (4 to 64
planes, chosen by the size of the launch) with L_tau that the depth divides
and does not divide, integers compared exactly with sums taken from the spins
on the host, for the batched pass (measurement sums and readings) and the
per-sample pass (spins after the exchange: lane sums over the slots)."""
import dataclasses

import numpy as np
import pytest

import qsg_workloads as W

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_2402_03920_amd import qsg  # noqa: E402


def lane_counts(words):
    bits = np.unpackbits(np.ascontiguousarray(words).view(np.uint8).reshape(-1, 8), axis=1,
                         bitorder="little")
    return bits.sum(axis=0, dtype=np.int64)


def host_sums(words, jx, jy, L, L_tau, anti):
    """(Bsp[64], Bt[64], q[32]) of one slot."""
    s = words.reshape(L_tau, L, L)
    V = s.size
    jx, jy = jx.reshape(L, L), jy.reshape(L, L)
    sp = lane_counts(s ^ np.roll(s, -1, axis=2) ^ jx) + lane_counts(s ^ np.roll(s, -1, axis=1) ^ jy)
    up = np.roll(s, -1, axis=0)
    if anti:
        up[-1] = ~up[-1]
    t = lane_counts(s ^ up)
    q = lane_counts(s ^ (s >> np.uint64(1)))[::2]
    return 2 * V - 2 * sp, V - 2 * t, V - 2 * q


# (L, L_tau, slots, samples): walks of 4, 8, 16, 32 and 64 planes at most,
# tiles of one and of two lengths
@pytest.mark.parametrize("L,L_tau,N,samples", [
    (2, 2, 3, 1), (6, 6, 3, 1), (6, 10, 3, 2), (4, 22, 5, 1), (16, 4, 2, 1),
    (6, 22, 32, 12), (10, 16, 40, 5), (12, 90, 24, 4), (18, 34, 34, 2),
    (16, 90, 48, 4), (16, 64, 48, 6), (24, 134, 48, 19)])
@pytest.mark.parametrize("anti", [False, True])
def test_walk_depths(L, L_tau, N, samples, anti):
    print(f"[energy] L={L} L_tau={L_tau} N={N} samples={samples} anti={anti}", flush=True)
    groups = [dataclasses.replace(
        W.tiny_group(L=L, L_tau=L_tau, beta=1.0, n_gamma=N, group_id=i, per_lane=True),
        antiperiodic=anti) for i in range(samples)]
    for flags in (qsg.QSG_BATCHED, qsg.QSG_PLAIN):
        with qsg.Ensemble(groups, pt_every=1, swaplog_cap=4) as ens:
            ens.init_spins()
            last = samples - 1
            jx, jy = ens.get_couplings(last)
            if flags == qsg.QSG_BATCHED:
                spins = ens.get_spins(last).reshape(N, -1)
                energies, overlaps = ens.energies()[last], ens.overlaps()[last]
                ens.pt_swap()
                sums = ens.sums()[last]
                for g in {0, N // 2, N - 1}:
                    sp, t, q = host_sums(spins[g], jx, jy, L, L_tau, anti)
                    assert np.array_equal(energies[g, :, 0], sp) and np.array_equal(energies[g, :, 1], t)
                    assert np.array_equal(overlaps[g], q)
                    assert np.array_equal(sums[g], np.concatenate([sp, t, q, q * q]))
            elif samples * N * L * L * L_tau < 6e6:
                ens.sweep(1, flags)
                spins, sums = ens.get_spins(last).reshape(N, -1), ens.sums()[last]
                sp, t = (sum(x) for x in list(zip(*(host_sums(w, jx, jy, L, L_tau, anti)
                                                    for w in spins)))[:2])
                assert np.array_equal(sums[:, :64].sum(axis=0), sp)
                assert np.array_equal(sums[:, 64:128].sum(axis=0), t)
