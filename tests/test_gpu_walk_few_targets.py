"""Few active particles, most in groups of their own: a longer list does not
take less time.  (Walked by whole workgroups, 900 groups took their 256
workgroups four rounds, 233 us, where 1150 groups took teams of four waves 135.)
The team's size does not change the sums: each row has the bits it has when the
same groups are walked in the other way."""
import numpy as np
import pytest
import torch

import workloads

pytestmark = pytest.mark.gpu
DEV = torch.device("cuda:0")


def test_few_targets(ag):
    n = 300000
    x, v, m = (torch.tensor(a, device=DEV) for a in workloads.plummer(n, seed=1))
    rng = np.random.default_rng(3)
    ms, groups = [], []
    with ag.Context(0) as c:
        c.tree_build(x, v, m, 16)
        for k in (1000, 1400):
            idx = torch.tensor(np.sort(rng.choice(n, k, replace=False)), dtype=torch.int32, device=DEV)
            f = [torch.zeros((n, q), dtype=torch.float64, device=DEV) for q in (3, 3, 6)]
            c.stats_reset()
            c.grav_eval(idx, 0.6, 0.01, 1.0, *f)
            groups.append(c.stats_read()["n_groups"])
            c.timing_enable(True)
            best = np.inf
            for _ in range(5):
                c.timing_read()
                for _ in range(10):
                    c.grav_eval(idx, 0.6, 0.01, 1.0, *f)
                best = min(best, c.timing_read()["walk"]["ms"])
            c.timing_enable(False)
            ms.append(best)
            # 64 waves per CU: four times as many workgroups before teams take over
            other = [torch.zeros_like(a) for a in f]
            c.set_option(ag.AG_OPT_WALK_WAVES_PER_CU, 64)
            c.grav_eval(idx, 0.6, 0.01, 1.0, *other)
            c.set_option(ag.AG_OPT_WALK_WAVES_PER_CU, 16)
            assert all(torch.equal(a, b) for a, b in zip(f, other))
    print(groups, ms)
    assert 256 < groups[0] < 1024 < groups[1]
    assert ms[0] < 1.2 * ms[1]
