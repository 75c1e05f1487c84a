"""The captured graph of colour passes and the same launches without a graph
against the oracle, bit for bit, on ensembles that one slot of more than
QSG_FUSED_GRAPH_WORDS words keeps from the fused chunk: small slots of unequal
shape, coupling ladders, antiperiodic prisms."""
from dataclasses import replace

import pytest

import qsg_workloads as W
from tests.parity_util import compare_state, oracle_groups

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_2402_03920_amd import qsg  # noqa: E402


def groups(anti):
    small = [(4, 8), (6, 4), (2, 2), (8, 6), (12, 10), (6, 2)]
    gs = [W.tiny_group(L=L, L_tau=Lt, beta=0.2 * Lt, n_gamma=1 + i, gmin=0.6, gmax=2.4, group_id=i,
                       per_lane=i % 2 == 1, j_seed=50 * i + 1) for i, (L, Lt) in enumerate(small)]
    gs += [W.tiny_k_group(L=4, L_tau=8, n_k=4, kmax=0.6, kmin=0.25, group_id=10),
           W.tiny_k_group(L=12, L_tau=10, n_k=5, kmax=0.35, kmin=0.27, group_id=12, j_seed=9),
           W.tiny_group(L=12, L_tau=18, beta=3.0, n_gamma=3, group_id=13)]  # 2592 words a slot
    return [replace(g, antiperiodic=anti and i != 0) for i, g in enumerate(gs)]


@pytest.mark.parametrize("anti", [False, True])
@pytest.mark.parametrize("flags", [qsg.QSG_BATCHED, qsg.QSG_BATCHED | qsg.QSG_GRAPH])
def test_colour_passes_follow_the_oracle(flags, anti):
    gs = groups(anti)
    assert max(g.L * g.L * g.L_tau for g in gs) > qsg.QSG_FUSED_GRAPH_WORDS
    print(f"[graph] flags={flags} anti={anti}", flush=True)
    ogs = oracle_groups(gs, 32)
    with qsg.Ensemble(gs, pt_every=5, swaplog_cap=32) as ens:
        ens.init_spins()
        for n in (7, 13, 20):  # whole chunks and remainders
            ens.sweep(n, flags)
            for og in ogs:
                og.run(n, 5)
            compare_state(ens, ogs)
