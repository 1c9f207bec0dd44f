"""Periodic walks by single waves and by teams of 4 give the same bits where the two
are written separately: nearest images, and Ewald sums of groups too wide for the
expansion about their centre (a single wave adds a tile's terms target by target, a
team a quarter of a tile's sixteenth at a time).  The second takes one target in each
of the 16^3 cells of the box: a parent of eight is cut into groups of 3, 3 and 2
neighbouring cells, whose extent is about two thirty-seconds of the box, the
expansion's limit."""
import numpy as np
import pytest
import torch

import workloads

pytestmark = pytest.mark.gpu
DEV = torch.device("cuda:0")


def _both(ag, x, v, m, ewald, cap, idx, waves):
    n = len(m)
    tx, tv, tm = (torch.tensor(a, device=DEV) for a in (x, v, m))
    ti = None if idx is None else torch.tensor(idx, dtype=torch.int32, device=DEV)
    got = []
    with ag.Context(0) as c:
        c.set_option(ag.AG_OPT_GROUP_TARGETS, cap)
        c.set_option(ag.AG_OPT_GROUP_SPAN, 0)
        c.set_periodic(1.0, ewald)
        c.tree_build(tx, tv, tm, 16)
        for w in waves:
            c.set_option(ag.AG_OPT_WALK_WAVES_PER_CU, w)
            f = [torch.zeros((n, k), dtype=torch.float64, device=DEV) for k in (3, 3, 6)]
            c.stats_reset()
            c.grav_eval(ti, 0.7, 1e-3, 1.0, *f)
            groups = c.stats_read()["n_groups"]
            got.append(f)
    for a, b in zip(*got):
        assert torch.equal(a, b)
    return groups


def test_nearest_images(ag):
    x, v, m = workloads.zeldovich_box(60, seed=6)
    groups = _both(ag, x, v, m, False, 10, None, (16, 64))   # four times as many waves: teams
    waves = torch.cuda.get_device_properties(0).multi_processor_count * 16
    assert 4 * waves < groups < 16 * waves


def test_wide_ewald_groups(ag):
    x, v, m = workloads.zeldovich_box(64, seed=6)
    cell = np.floor(x * 16).astype(int)
    away = np.abs(x * 16 - cell - 0.5).max(1)
    key = np.zeros(len(x), dtype=int)   # the cell's octal digits
    for b in range(4):
        for c in range(3):
            key |= ((cell[:, c] >> b) & 1) << (3 * b + 2 - c)
    order = np.lexsort((away, key))
    cells, first = np.unique(key[order], return_index=True)
    assert np.array_equal(cells, np.arange(4096))
    idx = order[first]                  # the particle nearest each cell's centre, in key order
    cuts = np.arange(4096).reshape(-1, 8)
    wide = 0
    for part in (cuts[:, :3], cuts[:, 3:6], cuts[:, 6:]):
        p = x[idx[part]]
        wide += int((((p.max(1) - p.min(1)) / 2).max(1) > 1.0 / 32).sum())
    print("wide groups:", wide)
    assert 300 < wide < 1236            # both kinds of group
    groups = _both(ag, x, v, m, True, 3, np.sort(idx), (1, 16))   # 256 waves: 1536 groups by single waves
    assert groups == 1536
