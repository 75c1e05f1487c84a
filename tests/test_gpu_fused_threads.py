"""Contexts of different slot sizes run their fused chunks from two threads at
once, each on a stream of its own, and follow the trajectory they have alone:
the kernel's limit of LDS serves both."""
import threading

import numpy as np
import pytest

import qsg_workloads as W

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_2402_03920_amd import qsg  # noqa: E402

SHAPES = [(16, 76), (10, 72)]  # 156 and 58 KiB of LDS


def run(L, L_tau, chunks, stream):
    g = W.tiny_group(L=L, L_tau=L_tau, beta=L_tau / 8.0, n_gamma=3, per_lane=True)
    with qsg.Ensemble([g], pt_every=2, swaplog_cap=4, stream=stream) as ens:
        ens.init_spins()
        for _ in range(chunks):  # a launch each, not a graph
            ens.sweep(2, qsg.QSG_BATCHED | qsg.QSG_FUSED)
        return ens.get_spins(0)


def test_two_threads_with_slots_of_different_size():
    streams = [torch.cuda.Stream() for _ in SHAPES]
    want = [run(*s, 60, st) for s, st in zip(SHAPES, streams)]
    got = [None, None]

    def work(i):
        got[i] = run(*SHAPES[i], 60, streams[i])

    threads = [threading.Thread(target=work, args=(i,)) for i in range(2)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    for a, b in zip(got, want):
        assert a is not None and np.array_equal(a, b)
