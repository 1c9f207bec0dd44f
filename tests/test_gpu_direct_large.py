"""The FP64 direct sum of many targets keeps 64 targets a workgroup where its
rounds of workgroups are as good as full: the sources are then summed in eight
subsets, as for a list of 16 384 targets (one round exactly), and the sums have
the same bits.  (Narrower tiles, whose workgroups stage every source as often
for fewer targets, took 20 % longer at both sizes; their sums differ in order.)"""
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
