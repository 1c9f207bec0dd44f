"""The tree build at the sizes where its kernels change: one workgroup sorts up
to 4096 particles in rows of 1024, the radix sort takes tiles of 1024, 2048 or 4096 and adds up
few tiles' counts itself, the inner levels run in one launch up to 8192
particles, and the nodes are counted by tiles of 512, 1024 or 2048 positions.
The tree is the oct-tree of the same particles on both sides of each edge.  The
moments are compared with extended-precision sums: the oracle adds one particle
after another in FP64, whose own error grows as n 1e-16 and passes the
comparison's 1e-12 at the larger sizes here."""
import numpy as np
import pytest
import torch

import workloads
from test_gpu_tree import _check_topology, _t

pytestmark = pytest.mark.gpu


class _Extended:
    @staticmethod
    def moments(x, v, m, rows):
        x, v, m = (np.asarray(a[rows], dtype=np.longdouble) for a in (x, v, m))
        M = m.sum()
        c, u = (m[:, None] * x).sum(0) / M, (m[:, None] * v).sum(0) / M
        y, w = x - c, v - u
        trace, cross = (m * (y * y).sum(1)).sum(), 2 * (m * (y * w).sum(1)).sum()
        ij = [(0, 0), (1, 1), (2, 2), (0, 1), (0, 2), (1, 2)]
        Q = [3 * (m * y[:, i] * y[:, j]).sum() - (trace if i == j else 0) for i, j in ij]
        Qd = [3 * (m * (y[:, i] * w[:, j] + w[:, i] * y[:, j])).sum() - (cross if i == j else 0) for i, j in ij]
        f = lambda a: np.asarray(a, dtype=np.float64)
        return {"M": float(M), "com": f(c), "u": f(u), "Q": f(Q), "Qdot": f(Qd), "lo": f(x.min(0)), "hi": f(x.max(0))}


@pytest.mark.parametrize("n", [2, 1024, 1025, 2049, 4096, 4097, 8192, 8193, 65536, 65537, 131073, 262144, 262145, (1 << 19) + 1,
                               (1 << 21) + 1])
def test_tree_at_edges(ctx, n):
    print(f"tree n={n}", flush=True)
    x, v, m = workloads.plummer(n, seed=n % 1000)
    ctx.tree_build(_t(x), _t(v), _t(m), 16)
    link, mom, perm = (t.cpu().numpy() for t in ctx.tree_export())
    _check_topology(link, mom, perm, n, 16, x, v, m, _Extended, sample=60)
    # a second build of the same particles is the same tree, bit for bit
    ctx.tree_build(_t(x), _t(v), _t(m), 16)
    for a, b in zip((link, mom, perm), ctx.tree_export()):
        assert torch.equal(torch.as_tensor(a), b.cpu())
