"""The FP64 direct sum of many targets keeps 64 targets a workgroup where its
rounds of workgroups are as good as full: the sources are then summed in eight
subsets, as for a list of 16 384 targets (one round exactly), and the sums have
the same bits.  (Narrower tiles, whose workgroups stage every source as often
for fewer targets, took 20 % longer at both sizes; their sums differ in order.)"""
import numpy as np
import pytest
import torch

import workloads

pytestmark = pytest.mark.gpu
DEV = torch.device("cuda:0")


@pytest.mark.parametrize("n", [30000, 300000])
def test_widest_tiles_for_many_targets(ag, n):
    print(f"direct n={n}", flush=True)
    x, v, m = (torch.tensor(a, device=DEV) for a in workloads.plummer(n, seed=5))
    idx = torch.arange(16384, dtype=torch.int32, device=DEV)
    with ag.Context(0) as c:
        out = []
        for rows in (None, idx):
            f = [torch.zeros((n, k), dtype=torch.float64, device=DEV) for k in (3, 3, 6)]
            c.grav_direct(x, v, m, rows, 0.01, 1.0, *f)
            out.append(f)
        c.sync()
    for a, b in zip(*out):
        assert torch.equal(a[:16384], b[:16384])


def test_rounding_of_long_sums(ag):
    """A lane's sums are taken in runs of 128 sources that are added up.  With random
    roundings of up to half an ulp at the size of the sum, growing evenly, a run of
    128 has an error of 2^-53 sqrt(128 / 9) of it (rms), the 30 runs of 30 000 sources in
    eight subsets another 2^-53 sqrt(30 / 9): 6e-16 together, of the diagonal sums of
    the tidal tensor, whose terms nearly cancel.  1.5e-15 of its norm leaves room for
    that and is passed twice over by one chain of all 3750 sources (4e-15)."""
    n = 30000
    x, v, m = workloads.plummer(n, seed=2)
    f = [torch.zeros((n, k), dtype=torch.float64, device=DEV) for k in (3, 3, 6)]
    with ag.Context(0) as c:
        c.grav_direct(*(torch.tensor(a, device=DEV) for a in (x, v, m)), None, 0.01, 1.0, *f)
        c.sync()
    t = f[2].cpu().numpy()
    x, m = x.astype(np.longdouble), m.astype(np.longdouble)
    w = np.array([1, 1, 1, 2, 2, 2])
    err = []
    for i in np.random.default_rng(0).choice(n, 100, replace=False):
        d = np.delete(x, i, 0) - x[i]
        mm, r2 = np.delete(m, i), (d * d).sum(1)
        if r2.min() < 1e-4:   # (softened pairs: another formula)
            continue
        f3 = mm / (r2 * np.sqrt(r2))
        ref = np.array([(f3 * ((3 * d[:, a] * d[:, b]) / r2 - (a == b))).sum()
                        for a, b in ((0, 0), (1, 1), (2, 2), (0, 1), (0, 2), (1, 2))])
        e = (t[i] - ref).astype(float)
        err.append((w * e * e).sum() / (w * ref.astype(float) ** 2).sum())
    print("rms", np.sqrt(np.mean(err)), len(err))
    assert np.sqrt(np.mean(err)) <= 1.5e-15
