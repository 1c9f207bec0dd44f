"""System offsets that are no partition of the particles are reported and read
nothing outside the arrays (they are kept within [0, n] before anything is read through
them); the context goes on with the next build."""
import numpy as np
import pytest
import torch

import workloads

pytestmark = pytest.mark.gpu
DEV = torch.device("cuda:0")


@pytest.mark.parametrize("off", [[0, 700, 1 << 40, 2100, 3000], [0, -(1 << 40), 1400, 2100, 3000], [0, 1400, 700, 2100, 3000],
                                 [0, 700, 1400, 2100, 2999], [1, 700, 1400, 2100, 3000], [0, 3000, 0, 3000, 3000]])
def test_bad_offsets_are_an_error(ag, off):
    print(off, flush=True)
    x, v, m = (torch.tensor(a, device=DEV) for a in workloads.plummer(3000, seed=2))
    f = [torch.zeros((3000, k), dtype=torch.float64, device=DEV) for k in (3, 3, 6)]
    with ag.Context(0) as c:
        c.tree_build_batched(x, v, m, torch.tensor(off, dtype=torch.int64, device=DEV), 16)
        with pytest.raises(ag.AgError) as e:
            c.sync()
        assert e.value.code == ag.AG_EDEVICE
        good = [0, 700, 1400, 2100, 3000]
        c.tree_build_batched(x, v, m, torch.tensor(good, dtype=torch.int64, device=DEV), 16)
        c.grav_eval_batched(None, 0.6, 0.01, 1.0, *f)
        c.sync()
    with ag.Context(0) as c:
        for a, b in zip(good, good[1:]):
            g = [torch.zeros((b - a, k), dtype=torch.float64, device=DEV) for k in (3, 3, 6)]
            c.tree_build(x[a:b].contiguous(), v[a:b].contiguous(), m[a:b].contiguous(), 16)
            c.grav_eval(None, 0.6, 0.01, 1.0, *g)
            c.sync()
            np.testing.assert_allclose(f[0][a:b].cpu(), g[0].cpu(), rtol=0, atol=1e-2 * float(g[0].abs().max()))
