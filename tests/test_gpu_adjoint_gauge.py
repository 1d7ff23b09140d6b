"""The reverse sweep's gauges, which each U half keeps of the iteration before it: the gradient with the whole
history kept (one segment), with segments of one iteration (every gauge from its own launch) and of three, for
rows of each row kernel, balanced and unbalanced; and a batch against its last pair alone."""

import math

import numpy as np
import pytest

import oracle as O

from helpers import announce, ensure_built, rel_l2, to_dev, to_np

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _built():
    ensure_built()


@pytest.mark.parametrize("precision,tol", [("fp32", 2e-4), ("fp64", 1e-9)])
@pytest.mark.parametrize("tau", [math.inf, 1.0])
@pytest.mark.parametrize("grid,pairs", [(("gl", 7, 1440, 7), 2), (("gl", 12, 180, 12), 2), (("gl", 130, 64, 20), 2),
                                        (("gl", 301, 24, 10), 1), (("gl", 5, 1999, 5), 1), (("hp", 17, 34), 2)])
def test_gauges_of_segments(grid, pairs, tau, precision, tol):
    from paper_2605_18389_amd import Plan
    announce(f"adjoint gauges {grid} x{pairs} tau={tau} {precision}")
    G = O.HealpixGrid(grid[1], grid[2]) if grid[0] == "hp" else O.make_grid(*grid)
    rng = np.random.default_rng(8)
    p, q = (0.5 + rng.random((pairs,) + tuple(G.field_shape)) for _ in range(2))
    P = Plan([grid], precision=precision, legendre="recurrence")
    pd, qd = to_dev(p, P.dtype), to_dev(q, P.dtype)
    S, g, _ = P.divergence_grad(pd, qd, 0.5, T=6, tau=tau)
    g = to_np(g).reshape(p.shape)
    for ck in (1, 3):
        Sk, gk, _ = P.divergence_grad(pd, qd, 0.5, T=6, tau=tau, checkpoint_every=ck)
        assert rel_l2(to_np(gk).reshape(p.shape), g) < tol
        np.testing.assert_allclose(np.asarray(Sk), np.asarray(S), rtol=0, atol=tol * max(1.0, np.abs(S).max()))
    i = pairs - 1
    _, g1, _ = P.divergence_grad(to_dev(p[i], P.dtype), to_dev(q[i], P.dtype), 0.5, T=6, tau=tau)
    assert rel_l2(g[i], to_np(g1).reshape(p[i].shape)) < tol
