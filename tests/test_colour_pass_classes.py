"""The colour pass numbers the classes of a slot by the ordering of its two
couplings (three regimes) and compares every level through the handler of the
slot's truth table at that level: every ladder has a regime, and slots of all
regimes and of extreme thresholds follow the oracle bit for bit."""
import numpy as np
import pytest

import qsg_workloads as W
from parity_util import compare_state, oracle_groups
from paper_2402_03920_amd import qsg

# classes (n_s, n_t) that may have dE > 0 in each regime: kp > 2k, k < kp <= 2k, kp <= k
REGIMES = ({(0, 0), (1, 0), (2, 0), (3, 0), (4, 0), (0, 1), (1, 1)},
           {(0, 0), (1, 0), (2, 0), (3, 0), (0, 1), (1, 1), (0, 2)},
           {(0, 0), (1, 0), (2, 0), (0, 1), (1, 1), (0, 2), (1, 2)})


def gamma_of(beta, L_tau, kp):
    """The field whose time coupling is kp."""
    return float(np.arctanh(np.exp(-2.0 * kp)) * L_tau / beta)


def live_classes(thr):
    return {(c // 3, c % 3) for c in range(15) if thr[c] != 0xFFFFFFFF}


def test_every_ladder_has_a_regime():
    rng = np.random.default_rng(17)
    rows = []
    for _ in range(60):
        L_tau = int(rng.choice([4, 32, 256, 2048]))
        beta = L_tau * float(np.exp(rng.uniform(np.log(1e-6), np.log(3.0))))
        k = beta / L_tau
        near = [gamma_of(beta, L_tau, f * k) for f in (2.0, 1.0)]  # on the regimes' borders
        for gamma in [*np.exp(rng.uniform(-12.0, 6.0, 6)), *near]:
            rows.append(qsg.qsg_build_tables(beta, L_tau, [gamma], cap=1)[0])
    for k in np.exp(rng.uniform(-16.0, 4.0, 40)):
        rows.append(qsg.qsg_build_tables_k([k], cap=1)[0])
    seen = set()
    for thr in np.concatenate(rows):
        fits = [i for i, r in enumerate(REGIMES) if live_classes(thr) <= r]
        assert fits
        seen.add(fits[0])
    assert seen == {0, 1, 2}


@pytest.mark.gpu
@pytest.mark.parametrize("form", ["plain", "batched", "fused"])
@pytest.mark.parametrize("k", [0.02, 0.5])
def test_regimes_follow_the_oracle(form, k):
    flags = {"plain": qsg.QSG_PLAIN, "batched": qsg.QSG_BATCHED,
             "fused": qsg.QSG_BATCHED | qsg.QSG_FUSED}[form]
    L_tau = 8
    # frozen, regime 0, 1, 1, 2, 2 and vanishing time coupling
    kps = [9.0, 2.6 * k, 1.9 * k, 1.1 * k, 0.9 * k, 0.2 * k]
    lad = np.array([gamma_of(k * L_tau, L_tau, kp) for kp in kps] + [400.0 / k])
    groups = [W.Group(4, L_tau, k * L_tau, lad, 0, 7, [1 + j for j in range(64)]),
              W.Group(6, L_tau, k * L_tau, lad[1:], 1, 8, [5] * 64, antiperiodic=True)]
    print(f"[colour] form={form} k={k}", flush=True)
    ogs = oracle_groups(groups, 16)
    with qsg.Ensemble(groups, pt_every=5, swaplog_cap=16, swap_table_cap=1 << 13) as ens:
        ens.init_spins()
        ens.sweep(30, flags)
        for og in ogs:
            og.run(30, 5)
        compare_state(ens, ogs)
