"""AG_OPT_WALK_WAVES_PER_CU over its whole range: every value gives the same
bits, and values below a workgroup's waves launch fewer workgroups (one wave per CU
is a sixteenth of the chip: at least four times as long; it was the same launch
as 16)."""
import numpy as np
import pytest
import torch

import workloads

pytestmark = pytest.mark.gpu
DEV = torch.device("cuda:0")


@pytest.mark.parametrize("adjoint", [False, True])
def test_every_value(ag, adjoint):
    n = 100000
    x, m, _ = workloads.uniform_sphere(n, seed=4)
    rng = np.random.default_rng(4)
    x, v, m, w = (torch.tensor(a, device=DEV) for a in (x, rng.normal(size=(n, 3)), m, rng.normal(size=(n, 3))))
    ms, first = {}, None
    with ag.Context(0) as c:
        c.tree_build(x, v, m, 16)
        c.timing_enable(True)
        for waves in (16, 1, 2, 4, 8, 11, 12, 15, 17, 32, 64):
            c.set_option(ag.AG_OPT_WALK_WAVES_PER_CU, waves)
            if adjoint:
                out = [torch.zeros_like(x), torch.zeros_like(m)]
                run = lambda: c.grav_backward(None, w, 0.7, 1e-3, 1.0, *out)   # noqa: E731
            else:
                out = [torch.zeros((n, k), dtype=torch.float64, device=DEV) for k in (3, 3, 6)]
                run = lambda: c.grav_eval(None, 0.7, 1e-3, 1.0, *out)          # noqa: E731
            run()
            c.timing_read()
            run()
            ms[waves] = c.timing_read()["adjoint" if adjoint else "walk"]["ms"]
            first = first or out
            assert all(torch.equal(a, b) for a, b in zip(first, out)), waves
    print(ms)
    assert ms[1] > 4.0 * ms[16]
