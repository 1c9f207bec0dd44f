"""The walk's particle lists: leaves of 1 to 300 particles in one place, around
the sizes at which the lists are written differently (8, 16 and 64 particles a
leaf) and beyond a list's 256 entries.  (Within 1e-9, not at one point: a leaf of
no extent is accepted as a node at any theta.)  At theta = 0 every target meets
every particle once: the number of pairs is n^2, and each target's g is the direct
sum's.  A missing or repeated particle moves a target by about 1/n of its
cancellation-free size (4e-4 here), the FP32 coordinates by 2^-24 2R / eps
(2e-6 at R <= 2, eps = 0.1): the bound is 1e-4."""
import numpy as np
import pytest

import workloads
from test_gpu_tree import _eval

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_leaf", [4, 16, 64])
def test_leaves_of_many_sizes(ctx, orc, n_leaf):
    rng = np.random.default_rng(5 + n_leaf)
    sizes = [1, 7, 8, 9, 15, 16, 17, 63, 64, 65, 255, 256, 257, 300, 2, 3]
    x = np.concatenate([rng.uniform(-1, 1, 3) + 1e-9 * rng.normal(size=(k, 3)) for k in sizes] + [rng.uniform(-1, 1, (1000, 3))])
    n = len(x)
    v, m = rng.normal(size=(n, 3)), rng.uniform(0.5, 1.5, n) / n
    ctx.stats_reset()
    a, j, t = _eval(ctx, x, v, m, 0.0, 0.1, n_leaf=n_leaf)
    st = ctx.stats_read()
    assert st["n_pp"] == n * n and st["n_pn"] == 0
    ar, _, _ = orc.direct(x, v, m, 0.1, 1.0)
    e = np.linalg.norm(a - ar, axis=1) / orc.abs_scale(x, m, 0.1, 1.0)
    print(f"n={n} n_leaf={n_leaf}: worst {e.max():.1e}", flush=True)
    assert e.max() <= 1e-4
