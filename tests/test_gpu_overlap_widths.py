"""Euclidean-time overlaps at every plane width and around the slices a wave
and a block take (4 and 32 up to L = 16, 2 and 16 above), integers compared
exactly with the oracle; fully ordered and checkerboard configurations give
the counters' extremes (all sites of a column equal or different)."""
import numpy as np
import pytest

import qsg_workloads as W
from oracle import overlaps

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_2402_03920_amd import qsg  # noqa: E402


def check(ens, L, L_tau, taus, n_slots):
    got = ens.tau_overlaps(0, range(n_slots), taus)
    spins = ens.get_spins(0).reshape(n_slots, -1)
    for s in range(n_slots):
        want = overlaps.contributions(spins[s], L, L_tau, taus)
        for key in ("q2", "q4", "A", "B"):
            assert np.array_equal(got[s][key], want[key]), (L, L_tau, s, key)


@pytest.mark.parametrize("L", range(2, 33, 2))
def test_widths_and_slice_counts(L):
    for L_tau in (2, 6, 18) if L > 20 else (2, 6, 18, 34, 38):
        print(f"[overlaps] L={L} L_tau={L_tau}", flush=True)
        g = W.tiny_group(L=L, L_tau=L_tau, beta=1.0, n_gamma=2, group_id=L, per_lane=True)
        with qsg.Ensemble([g], pt_every=5, swaplog_cap=4) as ens:
            ens.init_spins()
            ens.sweep(3, qsg.QSG_BATCHED)
            taus = sorted({0, 1, L_tau // 2, L_tau - 1})
            check(ens, L, L_tau, taus, 2)
            y, x = np.divmod(np.arange(L * L), L)
            tau = np.arange(L_tau)[:, None]
            board = np.where((x + y + tau) % 2, ~np.uint64(0), np.uint64(0xAAAAAAAA00000000))
            stripe = np.where(tau % 2, np.uint64(0), ~np.uint64(0)) | (np.uint64(1) << (x % 64).astype(np.uint64))
            words = np.concatenate([board.astype(np.uint64).ravel(),
                                    np.broadcast_to(stripe, (L_tau, L * L)).astype(np.uint64).ravel()])
            ens.set_spins(0, words)
            check(ens, L, L_tau, taus, 2)
