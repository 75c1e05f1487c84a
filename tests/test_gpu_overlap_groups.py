"""Overlaps of the smallest planes on launches of many blocks, where a wave
takes four groups of slices: around a block's 64 slices, integers equal to the
oracle's and to those of the same slots taken one by one (two groups)."""
import numpy as np
import pytest

import qsg_workloads as W
from oracle import overlaps

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_2402_03920_amd import qsg  # noqa: E402


@pytest.mark.parametrize("L,L_tau,N", [(2, 64, 8), (2, 130, 4), (2, 18, 12), (4, 66, 16), (4, 126, 10),
                                       (4, 34, 20)])
def test_many_blocks(L, L_tau, N):
    n = 64
    blocks = -(-L_tau // 32) * n * N
    assert blocks >= (512 if L == 2 else 2048)
    assert -(-L_tau // 32) * n < (512 if L == 2 else 2048)
    print(f"[overlaps] L={L} L_tau={L_tau} N={N}", flush=True)
    g = W.tiny_group(L=L, L_tau=L_tau, beta=L_tau / 16.0, n_gamma=N, gmin=2.0, gmax=4.0, per_lane=True)
    taus = [i % L_tau for i in range(n)]
    with qsg.Ensemble([g], pt_every=5, swaplog_cap=2) as ens:
        ens.init_spins()
        ens.sweep(5, qsg.QSG_BATCHED)
        got = ens.tau_overlaps(0, range(N), taus)
        spins = ens.get_spins(0).reshape(N, -1)
        for s in range(N):
            alone = ens.tau_overlaps(0, s, taus)[0]
            for key in ("q2", "q4", "A", "B"):
                assert np.array_equal(got[s][key], alone[key]), (s, key)
        for s in (0, N - 1):
            want = overlaps.contributions(spins[s], L, L_tau, taus)
            for key in ("q2", "q4", "A", "B"):
                assert np.array_equal(got[s][key], want[key]), (s, key)
