"""PT steps against the oracle, bit for bit, where their kernel can go wrong:
slot counts around the waves of its block (1 to 64), exchange tables from
empty over one entry to thousands, equal neighbours, both energies the
exchange weighs, and steps that follow sweeps, other steps and each other."""
import dataclasses

import numpy as np
import pytest

import qsg_workloads as W
from parity_util import compare_state, oracle_groups

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_2402_03920_amd import qsg  # noqa: E402


def ladder(N, kind):
    """Spacings from zero to wide, in turn."""
    steps = np.resize([0.0, 0.3, 0.004, 0.02, 0.06, 0.1], N - 1) if N > 1 else np.zeros(0)
    x = np.concatenate([[0.0], np.cumsum(steps)])
    return 0.01 * np.exp(x) if kind == "gamma" else 0.1 + 0.5 * x[::-1]


@pytest.mark.parametrize("kind", ["gamma", "k"])
@pytest.mark.parametrize("N", [1, 2, 15, 16, 17, 33, 64])
def test_pt_steps_bit_exact(N, kind):
    print(f"[pt] N={N} {kind}", flush=True)
    shapes = [(4, 6)] if N > 33 else [(4, 6), (8, 40)]
    groups = [dataclasses.replace(
        W.tiny_group(L=L, L_tau=L_tau, beta=1.0, n_gamma=N, group_id=7 + i, per_lane=True,
                     antiperiodic=i == 1),
        gammas=ladder(N, kind), ladder=kind) for i, (L, L_tau) in enumerate(shapes)]
    for flags in (qsg.QSG_BATCHED | qsg.QSG_GRAPH, qsg.QSG_PLAIN):
        ogs = oracle_groups(groups, log_cap=32)
        with qsg.Ensemble(groups, pt_every=2, swaplog_cap=32) as ens:
            ens.init_spins()
            ens.pt_swap()
            ens.sweep(5, flags)
            ens.pt_swap()
            ens.pt_swap()
            ens.sweep(6, flags)
            for og in ogs:
                og.pt_step()
                og.run(5, 2)
                og.pt_step()
                og.pt_step()
                og.run(6, 2)
            compare_state(ens, ogs)
