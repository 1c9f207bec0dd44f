"""A tree walk by single waves, by teams of 4 waves or by whole workgroups
(picked by the number of groups against the waves launched) gives the same
bits: teams evaluate the same tiles and fold their sums in the same order.
AG_OPT_WALK_WAVES_PER_CU moves the boundaries, so each case runs the same
groups two ways.  No tolerance: the results must be equal."""
import numpy as np
import pytest
import torch

import workloads

pytestmark = pytest.mark.gpu
DEV = torch.device("cuda:0")


def _t(a, dtype=None):
    return torch.tensor(a, device=DEV) if dtype is None else torch.tensor(a, dtype=dtype, device=DEV)


def _way(groups, waves_per_cu, team):
    """Which of the three ways the walk takes."""
    p = torch.cuda.get_device_properties(0).multi_processor_count * max(1, waves_per_cu // team) * team
    return "solo" if groups > 4 * p else ("small teams" if groups > p // 4 else "workgroup")


# (what, particles, targets per group, the two ways)
CASES = [("forward", 150001, 64, {"small teams", "workgroup"}), ("forward", 250007, 12, {"solo", "small teams"}),
         ("soft", 250007, 12, {"solo", "small teams"}), ("relative", 150001, 64, {"small teams", "workgroup"}),
         ("relative list", 150001, 64, {"small teams", "workgroup"}),
         ("near", 40 ** 3, 64, {"small teams", "workgroup"}),
         ("ewald", 44 ** 3, 64, {"small teams", "workgroup"}), ("ewald", 60 ** 3, 10, {"solo", "small teams"}),
         ("ewald wide", 64 ** 3, 64, {"small teams", "workgroup"}),
         ("adjoint", 100003, 64, {"small teams", "workgroup"}), ("adjoint", 200003, 12, {"solo", "small teams"})]


@pytest.mark.parametrize("what,n,targets,ways", CASES)
def test_same_bits_by_single_waves_and_teams(ag, what, n, targets, ways):
    rng = np.random.default_rng(n + targets)
    per = what in ("near", "ewald", "ewald wide")
    if per:
        x, v, m = workloads.zeldovich_box(round(n ** (1 / 3)), seed=6)
    else:
        x, m, _ = workloads.uniform_sphere(n, seed=2)
        v = rng.normal(size=x.shape)
    tx, tv, tm = _t(x), _t(v), _t(m)
    idx = None
    if what == "ewald wide":   # few targets in each group's cells: wide groups sum target by target
        idx = _t(workloads.random_subset(n, 0.3, seed=8).astype(np.int32), torch.int32)
    if what == "relative list":   # teams walk the groups of 40 000 targets or more in an order of their own
        idx = _t(workloads.random_subset(n, 0.5, seed=9).astype(np.int32), torch.int32)
    got, seen = [], set()
    with ag.Context(0) as c:
        c.set_option(ag.AG_OPT_GROUP_TARGETS, targets)
        if what == "soft":
            c.set_softening(_t(rng.uniform(0.5, 2.0, n) * n ** (-1 / 3)))
        if per:
            c.set_periodic(1.0, what != "near")
        c.tree_build(tx, tv, tm, 16)
        if what.startswith("relative"):
            c.set_relative_opening(0.0025, _t(-x))
        w = _t(rng.normal(size=x.shape))
        for waves in (16, 64):
            c.set_option(ag.AG_OPT_WALK_WAVES_PER_CU, waves)
            c.stats_reset()
            if what == "adjoint":
                out = [torch.zeros_like(tx), torch.zeros_like(tm)]
                c.grav_backward(None, w, 0.7, 1e-3, 1.0, *out)
                groups = c.stats_read()["n_groups"] // 2   # its forward walk and its adjoint walk
            else:
                out = [torch.zeros_like(tx), torch.zeros_like(tx), torch.zeros((n, 6), dtype=tx.dtype, device=DEV)]
                c.grav_eval(idx, 0.7, 1e-3, 1.0, *out)
                groups = c.stats_read()["n_groups"]
            got.append(out)
            seen.add(_way(groups, waves, 12 if what == "adjoint" else 16))
    assert seen == ways, (groups, seen)
    for a, b in zip(*got):
        assert torch.equal(a, b)


@pytest.mark.parametrize("n,targets", [(1, 64), (3001, 64), (150001, 64), (250007, 12)])
def test_tidal_tensor_alone(ag, n, targets):
    """The walk that sums the tidal tensor alone (whole workgroups, small teams,
    single waves) gives the bits of the one that also sums g and the jerk."""
    x, m, _ = workloads.uniform_sphere(n, seed=3)
    v = np.random.default_rng(n).normal(size=x.shape)
    with ag.Context(0) as c:
        c.set_option(ag.AG_OPT_GROUP_TARGETS, targets)
        c.tree_build(_t(x), _t(v), _t(m), 16)
        acc, jerk = (torch.zeros((n, 3), dtype=torch.float64, device=DEV) for _ in range(2))
        both, alone = (torch.zeros((n, 6), dtype=torch.float64, device=DEV) for _ in range(2))
        c.grav_eval(None, 0.7, 1e-3, 1.0, acc, jerk, both)
        c.grav_eval(None, 0.7, 1e-3, 1.0, None, None, alone)
    assert torch.equal(both, alone)
