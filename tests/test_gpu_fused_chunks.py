"""The fused chunk, also as the graph form takes it by itself for small slots,
gives the trajectory of one launch per sample and pass: words of a colour
around a wave, a block and several rounds of it, slots that just fit LDS or
do not, unequal groups, both ends of imaginary time."""
import numpy as np
import pytest

import qsg_workloads as W

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_2402_03920_amd import qsg  # noqa: E402

# (L, L_tau): 4 words up to 20 k
SHAPES = [(2, 2), (4, 8), (4, 10), (10, 20), (8, 32), (2, 514), (8, 40), (6, 72), (16, 24),
          (58, 2), (16, 76), (16, 78)]


def run(groups, flags):
    with qsg.Ensemble(groups, pt_every=3, swaplog_cap=4) as ens:
        ens.init_spins()
        ens.sweep(7, flags)   # two whole chunks and a remainder
        ens.sweep(5, flags)   # rest of the chunk, one more
        return ([ens.get_spins(i) for i in range(len(groups))], ens.sums(), ens.walkers(),
                ens.counters())


@pytest.mark.parametrize("shapes", [[s] for s in SHAPES] + [[(4, 8), (8, 40), (2, 2)],
                                                            [(16, 76), (4, 10), (6, 72)]])
@pytest.mark.parametrize("anti", [False, True])
def test_fused_equals_launches_per_pass(shapes, anti):
    print(f"[fused] {shapes} anti={anti}", flush=True)
    groups = [W.tiny_group(L=L, L_tau=Lt, beta=Lt / 8.0, n_gamma=3, group_id=i, per_lane=True,
                           antiperiodic=anti) for i, (L, Lt) in enumerate(shapes)]
    want = run(groups, qsg.QSG_PLAIN)
    for flags in (qsg.QSG_BATCHED | qsg.QSG_FUSED, qsg.QSG_BATCHED | qsg.QSG_GRAPH,
                  qsg.QSG_BATCHED | qsg.QSG_GRAPH | qsg.QSG_FUSED):
        got = run(groups, flags)
        assert got[3] == want[3] == (12, 4)
        for a, b in zip(got[:3], want[:3]):
            for x, y in zip(a, b):
                assert np.array_equal(x, y)
