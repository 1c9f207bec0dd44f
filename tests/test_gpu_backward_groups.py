"""The gradient of all rows groups its particles and orders the groups once, for
both of its walks; with a list each walk has its own.  (Phase "groups" counts one
launch for either.)"""
import numpy as np
import pytest
import torch

import workloads

pytestmark = pytest.mark.gpu
DEV = torch.device("cuda:0")


@pytest.mark.parametrize("listed,launches", [(False, 2), (True, 4)])
def test_one_grouping(ag, listed, launches):
    n = 100000
    x, m, _ = workloads.uniform_sphere(n, seed=5)
    x, m = (torch.tensor(a, device=DEV) for a in (x, m))
    w, gx, gm = torch.ones_like(x), torch.zeros_like(x), torch.zeros_like(m)
    idx = torch.tensor(np.arange(0, n, 2), dtype=torch.int32, device=DEV) if listed else None
    with ag.Context(0) as c:
        c.tree_build(x, torch.zeros_like(x), m, 16)
        c.timing_enable(True)
        c.grav_backward(idx, w, 0.7, 1e-3, 1.0, gx, gm)
        assert c.timing_read()["groups"]["launches"] == launches
