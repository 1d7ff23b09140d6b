"""Transforms alone and heat applies on both sides of the item counts from which the float64 batch kernel runs, for
each number of its latitude chunks, against the oracle."""

import numpy as np
import pytest

import oracle as O

from helpers import announce, ensure_built, rel_l2, to_dev, to_np

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _built():
    ensure_built()


@pytest.mark.parametrize("precision,tol", [("fp32", 1e-5), ("fp64", 1e-12)])
@pytest.mark.parametrize("grid,items", [(("gl", 100, 364, 181), 12), (("gl", 100, 364, 181), 13),
                                        (("gl", 380, 688, 344), 7), (("gl", 380, 688, 344), 12),
                                        (("gl", 380, 688, 344), 13), (("gl", 400, 700, 350), 7),
                                        (("gl", 400, 700, 350), 8), (("gl", 400, 700, 350), 17),
                                        (("gl", 520, 700, 350), 6), (("gl", 520, 700, 350), 8),
                                        (("gl", 650, 700, 350), 5), (("gl", 650, 700, 350), 6)])
def test_lines(grid, items, precision, tol):
    import torch
    from paper_2605_18389_amd import Plan
    announce(f"batch lines {grid} x{items} {precision}")
    G = O.make_grid(*grid)
    L = grid[-1]
    v = 0.5 + np.random.default_rng(1).random((items,) + tuple(G.field_shape))
    pick = [0, items - 1]
    P = Plan([grid], precision=precision, legendre="recurrence")
    out = to_np(P.heat_apply(to_dev(v, P.dtype), 1e-3)).reshape(v.shape)
    assert rel_l2(out[pick], O.heat_apply(v[pick], G, 1e-3)) < tol
    ref = np.concatenate(O.analysis(v[pick], G), axis=-1)
    got = P.analysis(to_dev(v, P.dtype)).detach().cpu().numpy().astype(np.complex128).reshape(items, -1)[pick]
    assert np.linalg.norm(got - ref) < tol * np.linalg.norm(ref)
    rng = np.random.default_rng(2)
    cs = [rng.standard_normal((items, L - m)) + 1j * (rng.standard_normal((items, L - m)) if m else 0)
          for m in range(L)]
    ct = torch.as_tensor(np.concatenate(cs, -1).reshape(-1), device="cuda")
    ct = ct.to(torch.complex128 if precision == "fp64" else torch.complex64)
    f = to_np(P.synthesis(ct)).reshape(v.shape)[pick]
    assert rel_l2(f, O.synthesis([c[pick] for c in cs], G)) < tol
