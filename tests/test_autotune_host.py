"""The autotuner's search, with a timer of the test's own: lanes are tried on the
levels that the timed launch takes by them, and no other level's change."""
import numpy as np
import torch

import gridgen
from paper_1811_02512_amd import api, autotune


def test_tail_levels_keep_their_lanes(monkeypatch):
    g = gridgen.make_grid(2000, 1)
    sym = api.Symbolic(g.n, g.f, g.t)
    before = sym.get_mapping().copy()
    tried = []

    class Timer:  # every run looks faster than the last: each trial is taken
        def __init__(self, *a):
            self.runs, self.ms = 0, 100.0

        def __call__(self):
            tried.append(sym.get_mapping().copy())
            self.runs += 1
            self.ms *= 0.98
            return self.ms

    monkeypatch.setattr(autotune, "_Timer", Timer)
    P = torch.zeros(4, g.n)
    res = autotune.tune(sym, None, None, P, P, P, P, passes=1, budgets=(65536,))
    below = sym.info.nlevels - sym.info.tail_levels
    assert 0 < below < sym.info.nlevels
    for m in tried + [np.asarray(res["mapping"]), sym.get_mapping()]:
        np.testing.assert_array_equal(m[below:], before[below:])
    # the levels below it are searched: every class of theirs changed
    assert not (np.asarray(res["mapping"])[:below] == before[:below]).any()
