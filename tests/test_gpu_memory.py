"""What calls fit in: a fresh context's buffers, with AG_OPT_MEM_LIMIT at sizes that
hold each sequence for 100 000 particles (bytes; a limit that has held a call goes on
holding it)."""
import pytest
import torch

pytestmark = pytest.mark.gpu
DEV = torch.device("cuda:0")
N = 100000
# n_leaf: build, evaluation, with a list, relative test, lengths, gradient, Ewald
FITS = {1: (468.10e6, 480.48e6, 479.04e6, 480.88e6, 480.48e6, 939.69e6, 483.36e6),
        16: (95.37e6, 100.01e6, 98.57e6, 100.41e6, 100.01e6, 194.27e6, 102.88e6),
        64: (58.67e6, 62.54e6, 61.10e6, 62.94e6, 62.54e6, 120.88e6, 65.42e6)}


@pytest.mark.parametrize("n_leaf", sorted(FITS))
def test_sequences_fit(ag, n_leaf):
    g = torch.Generator(device=DEV).manual_seed(1)
    x = torch.rand(N, 3, generator=g, device=DEV, dtype=torch.float64)
    v, m = torch.zeros_like(x), torch.full((N,), 1.0 / N, dtype=torch.float64, device=DEV)
    a, j, t = (torch.zeros((N, k), dtype=torch.float64, device=DEV) for k in (3, 3, 6))
    h = torch.zeros_like(m)
    idx = torch.arange(0, N, 10, device=DEV, dtype=torch.int32)

    def run(c, what):
        if what == "ewald":
            c.set_periodic(1.0, True)
        if what == "relative":
            c.set_relative_opening(0.01, torch.ones_like(x))
        c.tree_build(x, v, m, n_leaf)
        if what in ("eval", "relative", "ewald"):
            c.grav_eval(None, 0.6, 0.01, 1.0, a, j, t)
        elif what == "list":
            c.grav_eval(idx, 0.6, 0.01, 1.0, a, j, t)
        elif what == "lengths":
            c.neighbour_lengths(16, h)
        elif what == "gradient":
            c.grav_backward(None, a, 0.6, 0.01, 1.0, j, h)
        c.sync()

    for what, limit in zip(("build", "eval", "list", "relative", "lengths", "gradient", "ewald"), FITS[n_leaf]):
        with ag.Context(0) as c:
            c.set_option(ag.AG_OPT_MEM_LIMIT, int(limit))
            run(c, what)
