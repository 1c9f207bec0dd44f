"""The sorts rank lanes with equal digits by ballots, and each wave keeps its
counts per digit in LDS: all lanes of a digit read the count before one adds to
it.  Sets of few distinct positions put whole waves, rows and tiles on one digit,
or on two by turns; the permutation is then the rows by key, equal keys in row
order (n up to 4096 by one workgroup, above by tiles of 4, 8 and 16 rows of 64 a
wave)."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu
DEV = torch.device("cuda:0")


@pytest.mark.parametrize("n", [63, 64, 1025, 4096, 4097, 70001, 300001])
@pytest.mark.parametrize("cells", [1, 2, 7])
def test_rows_in_order(ctx, n, cells):
    rng = np.random.default_rng(n + cells)
    which = np.arange(n) % cells if cells < 7 else rng.integers(0, cells, n)
    # corners of the cube in key order (x the highest bit), so keys ascend with `which`
    corner = np.array([[(k >> 2) & 1, (k >> 1) & 1, k & 1] for k in range(8)], dtype=float)
    x = corner[which]
    t = lambda a: torch.tensor(a, device=DEV)   # noqa: E731
    for _ in range(3):
        ctx.tree_build(t(x), t(np.zeros_like(x)), t(np.full(n, 1.0 / n)), 16)
        perm = ctx.tree_export()[2].cpu().numpy()
        np.testing.assert_array_equal(perm, np.argsort(which, kind="stable"))
