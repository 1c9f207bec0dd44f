"""Price & Monaghan lengths that do not exist: where k particles coincide the sum
1 + sum w(r / h) of each is at least k at every h, so no length meets a target
below k.  The documented error comes back from the lists of 128 distances (four at a
point, n_ngb = 32: 4 against 3) and of 1024 (22 against 18.75) and from the steps of
eight targets (122 against 121.9, 1100 against 1031.25); the context goes on.

And supports of more particles than a list of 1024: 1100 others at about one distance
r of a target, of which 3 (1 + 2200 (1 - r / h)^3 = 3) bring h to 1.1 r.

And the time of long supports: it grows with the particles in them, not faster
(ten times as many at n_ngb 2000 as at 200 took 17 times as long with lists that
were cut again and again)."""
import numpy as np
import pytest
import torch

import workloads

pytestmark = pytest.mark.gpu
DEV = torch.device("cuda:0")


@pytest.mark.parametrize("n,k,n_ngb", [(700, 4, 32.0), (1500, 22, 200.0), (1500, 122, 1300.0), (3000, 1100, 11000.0)])
def test_no_length_is_an_error(ag, orc, n, k, n_ngb):
    print(f"pm n={n} coincident={k} n_ngb={n_ngb}", flush=True)
    x, _, m = workloads.plummer(n, seed=k)
    far = x.copy()
    x[5:5 + k] = x[5]
    with ag.Context(0) as c:
        for q, ok in ((x, False), (far, True), (x, False)):
            t = [torch.tensor(a, device=DEV) for a in (q, np.zeros_like(q), m)]
            c.tree_build(*t, 16)
            if ok:
                h, _ = c.pm_lengths(n_ngb)
                np.testing.assert_allclose(h.cpu().numpy(), orc.pm_lengths(q, n_ngb), rtol=1e-12, atol=0)
                continue
            with pytest.raises(ag.AgError, match="did not settle") as e:
                c.pm_lengths(n_ngb)
            assert e.value.code == ag.AG_EHIP


def test_support_beyond_every_list(ag, orc):
    rng = np.random.default_rng(4)
    d = rng.normal(size=(1100, 3))
    x = np.concatenate([np.zeros((1, 3)), d / np.linalg.norm(d, axis=1)[:, None] * rng.uniform(0.999, 1.001, (1100, 1))])
    t = [torch.tensor(a, device=DEV) for a in (x, np.zeros_like(x), np.full(len(x), 1.0 / len(x)))]
    with ag.Context(0) as c:
        c.tree_build(*t, 16)
        h, _ = c.pm_lengths(32.0)
    hr = orc.pm_lengths(x, 32.0)
    assert 1.05 < hr[0] < 1.15
    np.testing.assert_allclose(h.cpu().numpy(), hr, rtol=1e-12, atol=0)


def test_time_of_long_supports(ag):
    x, m, _ = workloads.uniform_sphere(100000, seed=3)
    t = [torch.tensor(a, device=DEV) for a in (x, np.zeros_like(x), m)]
    ms = []
    with ag.Context(0) as c:
        c.tree_build(*t, 16)
        for n_ngb in (200.0, 2000.0):
            c.pm_lengths(n_ngb)
            c.timing_enable(True)
            c.timing_read()
            for _ in range(3):
                c.pm_lengths(n_ngb)
            ms.append(c.timing_read()["neighbour"]["ms"])
            c.timing_enable(False)
    print(ms)
    assert ms[1] < 10.0 * ms[0]
