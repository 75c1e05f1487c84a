"""Readings of an ensemble of unequal groups (one launch for all of them)
equal the same groups read from ensembles of their own, for every kind, also
where a swap log is larger than the staging buffer (16 MiB) alone or only
together with its neighbours; state is unchanged by reading."""
import numpy as np
import pytest

import qsg_workloads as W

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_2402_03920_amd import qsg  # noqa: E402

KINDS = ("energies", "overlaps", "accepts", "walkers", "swaplog", "roundtrips", "sums", "histograms")


def readings(ens):
    return [[getattr(ens, k)() for k in KINDS] for _ in range(2)]


@pytest.mark.parametrize("slots,log_cap", [([1], 1), ([1, 64, 2, 3, 1, 17], 5),
                                           ([40, 2, 64], 40000), ([1] * 70, 3)])
def test_readings_of_unequal_groups(slots, log_cap):
    print(f"[readings] {slots[:6]} cap {log_cap}", flush=True)
    groups = [W.tiny_group(L=2 + 2 * (i % 3), L_tau=2 + 4 * (i % 2), beta=1.0, n_gamma=n,
                           group_id=i, per_lane=True) for i, n in enumerate(slots)]
    flags = qsg.QSG_BATCHED

    def run(gs):
        with qsg.Ensemble(gs, pt_every=2, swaplog_cap=log_cap) as ens:
            ens.init_spins()
            ens.sweep(8, flags)
            first, second = readings(ens)
            for a, b in zip(first, second):
                for x, y in zip(a, b):
                    assert np.array_equal(x, y)
            ens.sweep(2, flags)
            return first, [ens.get_spins(i) for i in range(len(gs))], ens.counters()

    got, spins, counters = run(groups)
    assert counters == (10, 5)
    for i, g in enumerate(groups):
        want, alone, _ = run([g])
        for k, a, b in zip(KINDS, got, want):
            assert np.array_equal(a[i], b[0]), (k, i)
        assert np.array_equal(spins[i], alone[0]), i
