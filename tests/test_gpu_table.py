"""Table plans' Legendre kernels (float32 and float64) against the oracle at the edges of their tiles: orders
below, at and above whole blocks of 32 rows, latitude pairs around multiples of 64 and up to the kernels' limit
of 512 and past it, and item counts around the 8 of a workgroup; heat apply, analysis and synthesis alone."""

import numpy as np
import pytest

import oracle as O

from helpers import announce, ensure_built, rel_l2, to_dev, to_np

pytestmark = pytest.mark.gpu

CASES = [(("gl", 2, 4, 1), 1), (("gl", 3, 8, 2), 9), (("gl", 31, 64, 31), 8), (("gl", 64, 64, 32), 7),
         (("gl", 33, 66, 33), 2), (("cc", 65, 128, 64), 17), (("gl", 127, 140, 65), 3), (("gl", 128, 72, 30), 1),
         (("gl", 129, 72, 30), 8), (("gl", 400, 80, 40), 9), (("gl", 769, 40, 20), 2), (("gl", 1024, 40, 20), 9),
         (("gl", 1026, 40, 20), 2)]


@pytest.fixture(scope="module", autouse=True)
def _built():
    ensure_built()


@pytest.mark.parametrize("precision,tol", [("fp32", 1e-5), ("fp64", 1e-12)])
@pytest.mark.parametrize("grid,items", CASES)
def test_table_kernels(grid, items, precision, tol):
    from paper_2605_18389_amd import Plan
    announce(f"table {grid} x{items} {precision}")
    G = O.make_grid(*grid)
    L = grid[3]
    v = 0.5 + np.random.default_rng(1).random((items, grid[1], grid[2]))
    P = Plan([grid], precision=precision, legendre="table")
    out = to_np(P.heat_apply(to_dev(v, P.dtype), 1e-3)).reshape(v.shape)
    assert rel_l2(out, O.heat_apply(v, G, 1e-3)) < tol
    c = P.analysis(to_dev(v, P.dtype))
    ref = np.concatenate(O.analysis(v, G), axis=-1)
    got = c.detach().cpu().numpy().astype(np.complex128).reshape(ref.shape)
    assert np.linalg.norm(got - ref) < tol * np.linalg.norm(ref)
    # synthesis of coefficients of every degree
    rng = np.random.default_rng(2)
    cs = [rng.standard_normal((items, L - m)) + 1j * (rng.standard_normal((items, L - m)) if m else 0)
          for m in range(L)]
    import torch
    ct = torch.as_tensor(np.concatenate(cs, -1).reshape(-1), device="cuda")
    ct = ct.to(torch.complex128 if precision == "fp64" else torch.complex64)
    f = to_np(P.synthesis(ct)).reshape(v.shape)
    assert rel_l2(f, O.synthesis(cs, G)) < tol
