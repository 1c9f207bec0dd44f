"""Lengths of few neighbours: the first radius holds them for every target of a run
in one traversal.  Right against the oracle for 1 to 16 neighbours, and one neighbour takes
clearly less time than eight (0.75 of it; 0.93 when nearly every run of targets
had one that found none and the run was traversed twice)."""
import numpy as np
import pytest
import torch

import workloads

pytestmark = pytest.mark.gpu
DEV = torch.device("cuda:0")


def _t(a):
    return torch.tensor(a, device=DEV)


@pytest.mark.parametrize("k", [1, 2, 7, 12, 13, 16])
def test_lengths(ag, orc, k):
    x, v, m = workloads.plummer(3001, seed=k)
    with ag.Context(0) as c:
        c.tree_build(_t(x), _t(v), _t(m), 16)
        h = c.neighbour_lengths(k)
        c.sync()
    np.testing.assert_array_equal(h.cpu().numpy(), orc.neighbour_length(x, k))


def test_time(ag):
    n = 1000000
    x = np.random.default_rng(1).uniform(-1, 1, (n, 3))
    ms = {}
    with ag.Context(0) as c:
        c.tree_build(_t(x), torch.zeros((n, 3), dtype=torch.float64, device=DEV), _t(np.full(n, 1.0 / n)), 16)
        h = torch.empty(n, dtype=torch.float64, device=DEV)
        c.timing_enable(True)
        for k in (1, 8):
            c.neighbour_lengths(k, h)
            ms[k] = np.inf
            for _ in range(5):
                c.timing_read()
                c.neighbour_lengths(k, h)
                ms[k] = min(ms[k], c.timing_read()["neighbour"]["ms"])
    print(ms)
    assert ms[1] < 0.83 * ms[8]
