"""Scans over more tiles than every tile adds up itself (8192: 2^24 rows or
positions, 2^21 nodes): due lists, the tree's node numbers, active lists and
groups at 2^24 + 3 particles, against the same lists made by torch and the
invariants of a pre-order tree; and the time of the due list, which grows with the
rows and not with their square."""
import pytest
import torch

pytestmark = pytest.mark.gpu
DEV = torch.device("cuda:0")


def _select(c, n, seed=1):
    g = torch.Generator(device=DEV).manual_seed(seed)
    tf = torch.zeros(n, dtype=torch.int64, device=DEV)
    bins = torch.where(torch.rand(n, generator=g, device=DEV) < 0.1, 10, 0).to(torch.int8)
    idx = torch.full((n,), -1, dtype=torch.int32, device=DEV)
    count = torch.zeros(1, dtype=torch.int64, device=DEV)
    c.adaptive_select(tf, bins, 1, 10, 0.5, idx, count)   # bin 10 (one tick) is due, bin 0 is not
    return bins, idx, count


def test_lists_and_tree(ag):
    n = (1 << 24) + 3
    g = torch.Generator(device=DEV).manual_seed(2)
    x = torch.rand(n, 3, generator=g, device=DEV, dtype=torch.float64)
    v = torch.zeros_like(x)
    m = torch.full((n,), 1.0 / n, dtype=torch.float64, device=DEV)
    with ag.Context(0) as c:
        bins, idx, count = _select(c, n)
        due = torch.nonzero(bins == 10).flatten()
        k = int(count)
        assert k == len(due) and torch.equal(idx[:k].long(), due) and bool((idx[k:] == -1).all())
        c.tree_build(x, v, m, 16)
        link, _, perm = c.tree_export()
        nn = link.shape[0]
        assert nn > 256 * 8192
        skip, start, cnt, lv = (link[:, q].long() for q in range(4))
        leaf = (lv & 0x100) != 0
        ids = torch.arange(nn, device=DEV)
        assert int(start[0]) == 0 and int(cnt[0]) == n and int(skip[0]) == nn
        assert torch.equal(skip[leaf], ids[leaf] + 1)
        ls, lc = start[leaf], cnt[leaf]
        assert int(ls[0]) == 0 and torch.equal(ls[1:], (ls + lc)[:-1]) and int(ls[-1] + lc[-1]) == n
        inner = ids[~leaf]
        end = torch.cat([start, torch.tensor([n], device=DEV)])[skip[inner]]
        assert torch.equal(start[inner + 1], start[inner]) and torch.equal(end, start[inner] + cnt[inner])
        assert torch.equal(perm.long().sort().values, torch.arange(n, device=DEV))
        acc = torch.zeros_like(x)
        c.stats_reset()
        c.grav_eval(idx[:k].contiguous(), 0.9, 1e-3, 1.0, acc, None, None)
        assert c.stats_read()["n_targets"] == k
        assert torch.equal((acc != 0).any(1), bins == 10)


def test_due_list_time_is_linear(ag):
    ms = []
    with ag.Context(0) as c:
        for lg in (27, 29):
            _select(c, 1 << lg)
            c.sync()
            c.timing_enable(True)
            for _ in range(3):
                _select(c, 1 << lg)
            ms.append(c.timing_read()["step"]["ms"])
            c.timing_enable(False)
    print(ms)
    # four times the rows: a factor of four, and one more for the runs' spread
    # (each tile adding up all before it: 7)
    assert ms[1] < 5.0 * ms[0]
