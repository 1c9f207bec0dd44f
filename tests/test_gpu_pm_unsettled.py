"""Price & Monaghan lengths that do not exist: where k particles coincide the sum
1 + sum w(r / h) of each is at least k at every h, so no length meets a target
below k.  The documented error comes back from the lists of 128 distances (four at a
point, n_ngb = 32: 4 against 3), of 1024 (122 against 121.9) and from the walk per step
beyond them (1100 against 1031.25); the context goes on."""
import numpy as np
import pytest
import torch

import workloads

pytestmark = pytest.mark.gpu
DEV = torch.device("cuda:0")


@pytest.mark.parametrize("n,k,n_ngb", [(700, 4, 32.0), (1500, 122, 1300.0), (3000, 1100, 11000.0)])
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
