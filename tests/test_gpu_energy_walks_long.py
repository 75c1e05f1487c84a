"""Bond sums of per-sample launches of 2^22 words and more, where the walks of
the energy pass have up to 32 and 64 planes: against the host's at 32, and
against the batched pass (checked against the host elsewhere) at 64.  Both
L_tau leave tiles of two lengths."""
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


def group(L_tau, anti):
    return dataclasses.replace(W.tiny_group(L=24, L_tau=L_tau, beta=1.0, n_gamma=48, per_lane=True),
                               antiperiodic=anti)


def stepped(g, flags):
    ens = qsg.Ensemble([g], pt_every=1, swaplog_cap=1)
    ens.init_spins()
    ens.sweep(1, flags)
    return ens


@pytest.mark.parametrize("anti", [False, True])
def test_walks_of_32_planes(anti):
    L, L_tau, N = 24, 154, 48
    print(f"[energy] L_tau={L_tau} anti={anti}", flush=True)
    assert N * L * L * L_tau >= 1 << 22
    with stepped(group(L_tau, anti), qsg.QSG_PLAIN) as ens:
        jx, jy = ens.get_couplings(0)
        sums = ens.sums()[0]
        rows = [host_sums(w, jx, jy, L, L_tau, anti) for w in ens.get_spins(0).reshape(N, -1)]
    # the exchange moves lanes between slots: lane sums over the slots stay
    for k in range(2):
        assert np.array_equal(sums[:, 64 * k:64 * k + 64].sum(axis=0), sum(r[k] for r in rows))


@pytest.mark.parametrize("anti", [False, True])
def test_walks_of_64_planes(anti):
    L_tau = 2430
    print(f"[energy] L_tau={L_tau} anti={anti}", flush=True)
    assert 48 * 24 * 24 * L_tau >= 1 << 26
    got = []
    for flags in (qsg.QSG_PLAIN, qsg.QSG_BATCHED):
        with stepped(group(L_tau, anti), flags) as ens:
            got.append((ens.sums()[0], ens.walkers()[0]))
    assert np.array_equal(got[0][0], got[1][0]) and np.array_equal(got[0][1], got[1][1])
