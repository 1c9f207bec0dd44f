"""The near-neighbour kernels where their lists are cut, emptied or given up:
more equal and near-equal distances than a length list holds (k + 64), supports
beyond the density solve's 128- and 1024-entry lists, sums over more than 128
neighbours, and runs of one target.  Against the oracle: lengths bit for bit;
h, Omega, Z and the correction within the bounds of a sum of at most n FP64
terms in another order (n 2^-53 < 2e-13 here) and the solve's 2e-14, taken as
1e-12 of h, of 1, and of the largest |Z| and |a|."""
import numpy as np
import pytest
import torch

import workloads

pytestmark = pytest.mark.gpu
DEV = torch.device("cuda:0")


def _t(a):
    return torch.tensor(a, device=DEV)


def _build(c, x, m, h=None):
    c.set_softening(None if h is None else _t(h))
    c.tree_build(_t(x), _t(np.zeros_like(x)), _t(m), 16)


@pytest.mark.parametrize("box", [0.0, 1.0])
@pytest.mark.parametrize("k", [1, 63, 64])
def test_lengths_cut_lists(ag, orc, k, box):
    rng = np.random.default_rng(k)
    same = np.tile(rng.uniform(0.2, 0.8, (1, 3)), (300, 1))             # 299 zeros before any other
    g = np.stack(np.meshgrid(*[np.arange(9) / 64.0] * 3, indexing="ij"), -1).reshape(-1, 3)
    core = 0.5 + 1e-4 * rng.normal(size=(900, 3))                       # a dense core inside a thin halo
    x = np.concatenate([same, g, core, rng.uniform(0.0, 1.0, (250, 3))])
    for targets in (64, 1):
        with ag.Context(0) as c:
            c.set_option(ag.AG_OPT_GROUP_TARGETS, targets)
            if box:
                c.set_periodic(box)
            _build(c, x, np.full(len(x), 1.0 / len(x)))
            h = c.neighbour_lengths(k)
            c.sync()
        np.testing.assert_array_equal(h.cpu().numpy(), orc.neighbour_length(x, k, box=box) if box
                                      else orc.neighbour_length(x, k))


@pytest.mark.parametrize("n_ngb,targets", [(32.0, 1), (140.0, 64), (1300.0, 64)])
def test_long_lists(ag, orc, n_ngb, targets):
    x, _, m = workloads.plummer(1500, seed=41)
    hr = orc.pm_lengths(x, n_ngb)
    omr, zr = orc.pm_terms(x, m, hr, n_ngb, 1.0)
    ar = orc.pm_correction(x, m, hr, n_ngb, 1.0)
    with ag.Context(0) as c:
        c.set_option(ag.AG_OPT_GROUP_TARGETS, targets)
        _build(c, x, m)
        h, om = c.pm_lengths(n_ngb)
        _build(c, x, m, hr)
        z = c.pm_factors(n_ngb, 1.0, _t(omr))
        a = c.pm_correct(_t(zr))
        c.sync()
    np.testing.assert_allclose(h.cpu().numpy(), hr, rtol=1e-12, atol=0)
    np.testing.assert_allclose(om.cpu().numpy(), omr, rtol=0, atol=1e-12 * max(1.0, np.abs(omr).max()))
    np.testing.assert_allclose(z.cpu().numpy(), zr, rtol=0, atol=1e-12 * np.abs(zr).max())
    np.testing.assert_allclose(a.cpu().numpy(), ar, rtol=0, atol=1e-12 * np.abs(ar).max())
