"""A pair's jerk enters the FP64 direct sum with one rounding at the size of the
sum.  Eight sources at distances 2 .. 4 on the z axis, one for each of the
eight subsets a workgroup of 64 targets sums separately, give the target at the
origin sums j_y of 1/2 to 1 in each (an ulp is 2^-53).  Every other source lies on
the line x = y at d = (a, a, 0) with velocity (b, -3 b - e, 0) and adds
m f nu_y + m D (d.nu) d_y = m f e / 2 to j_y, a difference of two terms of 3 b m f.  With
m f <= 2^-12 and e = 0.6 2^-41 that is at most 0.3 ulps, and the rounding of its terms
(about 20 2^-53 m f |nu| <= 2^-59) leaves it below the half ulp that a sum rounded once
drops: j_y has the bits of the same call with those masses zero.  (Added term by
term, the first term's rounding at the sum's size carries a pair in three over.)"""
import numpy as np
import pytest

from test_gpu_direct import _run_direct

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("soft,box", [(False, 0.0), (True, 0.0), (False, 100.0)])
def test_one_rounding_per_pair(ag, soft, box):
    import torch
    n = 16384
    rng = np.random.default_rng(3)
    x, v, m = np.zeros((n, 3)), np.zeros((n, 3)), np.empty(n)
    x[:8, 2] = np.linspace(2.0, 4.0, 8)
    m[:8] = 2.0
    v[:8, 1] = rng.uniform(0.25, 0.5, 8) * x[:8, 2] ** 3      # j_y = m v / r^3 = 0.5 .. 1
    a = rng.uniform(0.5, 2.0, n - 8)
    x[8:, 0] = x[8:, 1] = a
    b = rng.integers(2 ** 18, 2 ** 20, n - 8) * 2.0 ** -20
    v[8:, 0], v[8:, 1] = b, -3.0 * b - 0.6 * 2.0 ** -41
    m[8:] = rng.uniform(0.7, 1.0, n - 8) * 2.0 ** -12 * a ** 3 * 2.0 ** 1.5
    x[-1], v[-1], m[-1] = 0.0, 0.0, 2.0 ** -40                # the target
    out = []
    for with_line in (True, False):
        mm = m.copy()
        mm[1024 if with_line else 8:] = 0.0   # (one staged tile, in which the sums are one chain)
        with ag.Context(0) as c:
            if soft:
                c.set_softening(torch.full((n,), 1e-3, dtype=torch.float64, device="cuda:0"))
            if box:
                c.set_periodic(box)
            _, j, _ = _run_direct(ag, c, x, v, mm, 1e-3, 1.0, ag.AG_FP64)
        out.append(j[-1, 1])
    assert 4.0 < out[1] < 8.0
    assert out[0] == out[1]
