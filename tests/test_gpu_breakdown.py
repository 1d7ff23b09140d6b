"""The iteration of an item's breakdown on each form of the row launches, in a batch where only some items break
down, over many iterations after it (every later half is bad as well)."""

import numpy as np
import pytest

import oracle as O

from helpers import announce, ensure_built, to_dev

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _built():
    ensure_built()


@pytest.mark.parametrize("precision", ["fp32", "fp64"])
@pytest.mark.parametrize("grid,items", [(("gl", 32, 64, 32), 3), (("gl", 45, 180, 44), 4), (("gl", 45, 180, 44), 48),
                                        (("gl", 41, 202, 30), 3), (("gl", 12, 1440, 12), 3), (("hp", 16, 32), 3)])
def test_first_breakdown(grid, items, precision):
    from paper_2605_18389_amd import Plan
    announce(f"first breakdown {grid} x{items} {precision}")
    G = O.HealpixGrid(grid[1], grid[2]) if grid[0] == "hp" else O.make_grid(*grid)
    rng = np.random.default_rng(1)
    p, q = (0.9 + 0.2 * rng.random((items,) + tuple(G.field_shape)) for _ in range(2))
    # odd items: q all but vanishes outside a band of rows, at a heat time too short for the band limit, whose
    # kernel is negative there
    P = Plan([grid], precision=precision, legendre="recurrence")
    x = P.pixel_coords(0)[0]
    tiny = 1e-30 if precision == "fp32" else 1e-200
    q[1::2] = np.where((np.abs(x) < 0.5).reshape(G.field_shape), q[1::2], tiny)
    eps = [1e-4 if i % 2 else 1.0 for i in range(items)]
    ref = O.sinkhorn(p[1], q[1], G, 1e-4, T=2)
    assert ref["breakdown"] == 2
    pd, qd = to_dev(p, P.dtype), to_dev(q, P.dtype)
    for T in (2, 40):
        info = P.sinkhorn(pd, qd, eps, T=T)[2]
        assert [v["breakdown_iter"] for v in info] == [2 * (i % 2) for i in range(items)]
