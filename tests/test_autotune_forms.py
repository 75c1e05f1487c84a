"""The forms the tuner times are the forms the library runs: a graph of small
slots holds the fused chunk whichever flag asks for it, so there is one form
and nothing to pick by noise."""
import os
import re
import types

import qsg_workloads as W
from paper_2402_03920_amd import autotune, qsg

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


class Recorder:
    def __init__(self, shapes):
        self.groups = [W.tiny_group(L=L, L_tau=Lt, group_id=i) for i, (L, Lt) in enumerate(shapes)]
        self.cfg = types.SimpleNamespace(pt_every=10)
        self.stream = None
        self.flags = set()

    def sweep(self, n, flags):
        self.flags.add(flags)


def test_the_limit_is_the_header_s():
    text = open(os.path.join(ROOT, "include", "qsg.h")).read()
    assert int(re.search(r"#define QSG_FUSED_GRAPH_WORDS (\d+)u", text).group(1)) == \
        qsg.QSG_FUSED_GRAPH_WORDS


def test_small_slots_have_one_form(monkeypatch):
    monkeypatch.setattr(autotune, "_timer", lambda stream: lambda fn: (fn(), 1.0)[1])
    at_limit = [(8, 40), (4, 8)]  # 2560 words and fewer
    over = [(4, 8), (2, 642)]     # one slot of 2568
    name, flags, times = autotune.pick_form(Recorder(at_limit))
    assert (name, flags, list(times)) == ("fused", autotune.FORMS["fused"], ["fused"])
    ens = Recorder(over)
    assert set(autotune.pick_form(ens)[2]) == {"per-pass", "fused"}
    assert ens.flags == set(autotune.FORMS.values())
