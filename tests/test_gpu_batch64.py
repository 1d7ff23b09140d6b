"""Recurrence plans' float64 matrix-core Legendre kernel (batches) against the oracle at the edges of its tiles:
orders below, at and above whole blocks of 32 rows, latitude pairs around multiples of 64 and up to the kernel's
limit of 384 and past it, item counts around whole workgroups of 8 and on both sides of the rule that chooses it;
heat apply, analysis and synthesis alone, a batch of two interleaved grids, and a replayed solve."""

import math

import numpy as np
import pytest

import oracle as O

from helpers import announce, ensure_built, rel_l2, to_dev, to_np

pytestmark = pytest.mark.gpu

CASES = [(("gl", 31, 64, 31), 67), (("gl", 32, 64, 32), 64), (("gl", 32, 64, 32), 62), (("gl", 33, 66, 33), 63),
         (("cc", 65, 128, 64), 33), (("gl", 127, 140, 65), 32), (("gl", 129, 80, 40), 52), (("gl", 130, 80, 40), 57),
         (("gl", 200, 402, 200), 11), (("gl", 200, 402, 200), 10), (("gl", 400, 80, 40), 52),
         (("gl", 768, 40, 20), 104), (("gl", 769, 40, 20), 104), (("gl", 720, 1440, 720), 5), (("hp", 20, 40), 55),
         (("gl", 9, 16, 1), 2050)]


@pytest.fixture(scope="module", autouse=True)
def _built():
    ensure_built()


def _oracle_grid(g):
    return O.HealpixGrid(g[1], g[2]) if g[0] == "hp" else O.make_grid(*g)


@pytest.mark.parametrize("precision,tol", [("fp32", 1e-5), ("fp64", 1e-12)])
@pytest.mark.parametrize("grid,items", CASES)
def test_batch_kernel(grid, items, precision, tol):
    import torch
    from paper_2605_18389_amd import Plan
    announce(f"batch {grid} x{items} {precision}")
    G = _oracle_grid(grid)
    L = grid[-1]
    v = 0.5 + np.random.default_rng(1).random((items,) + tuple(G.field_shape))
    pick = sorted({0, items // 2, items - 1})
    P = Plan([grid], precision=precision, legendre="recurrence")
    out = to_np(P.heat_apply(to_dev(v, P.dtype), 1e-3)).reshape(v.shape)
    assert rel_l2(out[pick], O.heat_apply(v[pick], G, 1e-3)) < tol
    ref = np.concatenate(O.analysis(v[pick], G), axis=-1)
    got = P.analysis(to_dev(v, P.dtype)).detach().cpu().numpy().astype(np.complex128).reshape(items, -1)[pick]
    assert np.linalg.norm(got - ref) < tol * np.linalg.norm(ref)
    # synthesis of coefficients of every degree
    rng = np.random.default_rng(2)
    cs = [rng.standard_normal((items, L - m)) + 1j * (rng.standard_normal((items, L - m)) if m else 0)
          for m in range(L)]
    ct = torch.as_tensor(np.concatenate(cs, -1).reshape(-1), device="cuda")
    ct = ct.to(torch.complex128 if precision == "fp64" else torch.complex64)
    f = to_np(P.synthesis(ct)).reshape(v.shape)[pick]
    assert rel_l2(f, O.synthesis([c[pick] for c in cs], G)) < tol


@pytest.mark.parametrize("precision,tol", [("fp32", 1e-5), ("fp64", 1e-12)])
def test_batch_of_two_grids(precision, tol):
    from paper_2605_18389_amd import Plan
    grids = [("gl", 64, 130, 64), ("hp", 32, 64)]
    announce(f"batch of two grids {precision}")
    gs = [_oracle_grid(g) for g in grids]
    n = 66
    goi = [i & 1 for i in range(n)]
    rng = np.random.default_rng(3)
    fields = [0.5 + rng.random(tuple(gs[k].field_shape)) for k in goi]
    t = 10.0 ** rng.uniform(-4, -1, n)
    P = Plan(grids, precision=precision, legendre="recurrence")
    out = to_np(P.heat_apply(to_dev(np.concatenate([f.ravel() for f in fields]), P.dtype), t, grid_of_item=goi))
    off = 0
    for i, k in enumerate(goi):
        m = fields[i].size
        if i in (0, 1, 17, 32, 64, 65):
            ref = O.heat_apply(fields[i], gs[k], t[i])
            assert rel_l2(out[off:off + m].reshape(ref.shape), ref) < tol
        off += m


@pytest.mark.parametrize("precision,tol", [("fp32", 1e-4), ("fp64", 1e-10)])
@pytest.mark.parametrize("tau", [math.inf, 1.0])
def test_batch_solve(tau, precision, tol):
    """A solve of more items than the rule's line, run twice (its steps replay from a graph)."""
    from paper_2605_18389_amd import Plan
    announce(f"batch solve tau={tau} {precision}")
    grid, n = ("gl", 64, 128, 64), 40
    G = _oracle_grid(grid)
    rng = np.random.default_rng(5)
    p, q = 0.5 + rng.random((n, 64, 128)), 0.5 + rng.random((n, 64, 128))
    P = Plan([grid], precision=precision, legendre="recurrence")
    pick = [0, 20, 39]
    r = O.sinkhorn(p[pick], q[pick], G, 0.5, tau, T=4, C=2)
    for _ in range(2):
        phi, psi, info = P.sinkhorn(to_dev(p, P.dtype), to_dev(q, P.dtype), 0.5, tau, T=4, C=2)
        assert rel_l2(to_np(phi).reshape(p.shape)[pick], r["phi"]) < tol
        assert rel_l2(to_np(psi).reshape(p.shape)[pick], r["psi"]) < tol
        for k, i in enumerate(pick):
            assert info[i]["status"] == 0
            assert abs(info[i]["cost"] - r["cost"][k]) <= tol * abs(r["cost"][k])
