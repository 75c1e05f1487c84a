"""Bond sums and overlaps of the energy pass where slots of many columns or
planes ask for walks deeper than the words of the launch do (tiles of one and
two lengths), and where 64 planes are read ahead on fewer than 2^26 words:
integers equal to the host's, for the batched and the per-sample pass."""
import dataclasses

import numpy as np
import pytest

import qsg_workloads as W

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_2402_03920_amd import qsg  # noqa: E402
from tests.test_gpu_energy_walks import host_sums  # noqa: E402


@pytest.mark.parametrize("L,L_tau,N,samples", [
    (24, 2048, 1, 1), (24, 2046, 2, 1), (16, 2048, 2, 1), (64, 64, 12, 1), (256, 2, 2, 1),
    (130, 10, 3, 1), (2, 65536, 2, 1), (16, 128, 32, 7), (20, 96, 34, 5)])
def test_deep_walks(L, L_tau, N, samples):
    print(f"[energy] L={L} L_tau={L_tau} N={N} samples={samples}", flush=True)
    groups = [dataclasses.replace(
        W.tiny_group(L=L, L_tau=L_tau, beta=L_tau / 16.0, n_gamma=N, gmin=2.0, gmax=4.0, group_id=i,
                     per_lane=True), antiperiodic=i == 0) for i in range(samples)]
    for flags in (qsg.QSG_BATCHED, qsg.QSG_PLAIN):
        with qsg.Ensemble(groups, pt_every=1, swaplog_cap=1, swap_table_cap=1 << 16) as ens:
            ens.init_spins()
            jx, jy = ens.get_couplings(0)
            if flags == qsg.QSG_BATCHED:
                spins = ens.get_spins(0).reshape(N, -1)
                energies, overlaps = ens.energies()[0], ens.overlaps()[0]
                for g in {0, N - 1}:
                    sp, t, q = host_sums(spins[g], jx, jy, L, L_tau, True)
                    assert np.array_equal(energies[g, :, 0], sp)
                    assert np.array_equal(energies[g, :, 1], t) and np.array_equal(overlaps[g], q)
            else:
                ens.sweep(1, flags)
                spins, sums = ens.get_spins(0).reshape(N, -1), ens.sums()[0]
                rows = [host_sums(w, jx, jy, L, L_tau, True) for w in spins]
                # the exchange moves lanes between slots: sums over the slots stay
                for k in range(2):
                    assert np.array_equal(sums[:, 64 * k:64 * k + 64].sum(axis=0),
                                          sum(r[k] for r in rows))
