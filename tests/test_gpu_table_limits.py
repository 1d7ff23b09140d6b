"""Float64 tables at the limit of their matrix-core kernel, 448 latitude pairs, and past it (the vector-unit kernel),
against the oracle; one and several items, every mode."""

import numpy as np
import pytest

import oracle as O

from helpers import announce, ensure_built, rel_l2, to_dev, to_np

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _built():
    ensure_built()


@pytest.mark.parametrize("items", [1, 9])
@pytest.mark.parametrize("nlat", [895, 896, 897, 898])
def test_float64_table_limit(nlat, items):
    import torch
    from paper_2605_18389_amd import Plan
    announce(f"float64 table of {nlat} rows x{items}")
    grid, L = ("gl", nlat, 70, 35), 35
    G = O.make_grid(*grid)
    v = 0.5 + np.random.default_rng(1).random((items, nlat, 70))
    P = Plan([grid], precision="fp64", legendre="table")
    assert rel_l2(to_np(P.heat_apply(to_dev(v, P.dtype), 1e-3)).reshape(v.shape), O.heat_apply(v, G, 1e-3)) < 1e-12
    ref = np.concatenate(O.analysis(v, G), axis=-1)
    got = P.analysis(to_dev(v, P.dtype)).cpu().numpy().reshape(ref.shape)
    assert np.linalg.norm(got - ref) < 1e-12 * np.linalg.norm(ref)
    rng = np.random.default_rng(2)
    cs = [rng.standard_normal((items, L - m)) + 1j * (rng.standard_normal((items, L - m)) if m else 0)
          for m in range(L)]
    ct = torch.as_tensor(np.concatenate(cs, -1).reshape(-1), device="cuda")
    assert rel_l2(to_np(P.synthesis(ct)).reshape(v.shape), O.synthesis(cs, G)) < 1e-12
