"""Heat applies of the row-split recurrence kernel against the oracle on both sides of its one-pass forms: latitude
pairs around 64, 128 and 192, orders of fewer rows than a block, of whole blocks and one more, orders cut into
several parts, one item and pairs of items with one left over, and the operator's symmetry between the two modes."""

import numpy as np
import pytest

import oracle as O

from helpers import announce, ensure_built, rel_l2, to_dev, to_np

pytestmark = pytest.mark.gpu

GRIDS = [("gl", 2, 4, 1), ("gl", 128, 36, 17), ("gl", 130, 20, 8), ("cc", 129, 256, 128), ("gl", 256, 68, 33),
         ("gl", 257, 64, 32), ("gl", 384, 98, 48), ("gl", 385, 98, 49), ("gl", 386, 30, 15), ("gl", 376, 752, 376),
         ("hp", 24, 47)]


@pytest.fixture(scope="module", autouse=True)
def _built():
    ensure_built()


@pytest.mark.parametrize("precision,tol", [("fp32", 1e-5), ("fp64", 1e-12)])
@pytest.mark.parametrize("grid", GRIDS)
def test_one_pass_heat(grid, precision, tol):
    from paper_2605_18389_amd import Plan
    announce(f"one pass {grid} {precision}")
    G = O.HealpixGrid(grid[1], grid[2]) if grid[0] == "hp" else O.make_grid(*grid)
    P = Plan([grid], precision=precision, legendre="recurrence")
    for items in (1, 2, 3):
        v = 0.5 + np.random.default_rng(items).random((items,) + tuple(G.field_shape))
        for tr in (False, True):
            out = to_np(P.heat_apply(to_dev(v, P.dtype), 1e-3, transpose=tr)).reshape(v.shape)
            assert rel_l2(out, O.heat_apply(v, G, 1e-3, transpose=tr)) < tol
        # the same operator from its two halves: analysis and synthesis alone take two launches
        if items == 2:
            one = to_np(P.heat_apply(to_dev(v, P.dtype), 0.0)).reshape(v.shape)
            two = to_np(P.synthesis(P.analysis(to_dev(v, P.dtype)))).reshape(v.shape)
            assert rel_l2(one, two) < tol
