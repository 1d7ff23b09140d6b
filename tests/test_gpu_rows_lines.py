"""Row transforms on both sides of the lines between their launch forms, against the oracle: heat applies, solves and
gradients of few and many row pairs, balanced and unbalanced."""

import math

import numpy as np
import pytest

import oracle as O

from helpers import announce, ensure_built, rel_l2, to_dev, to_np

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _built():
    ensure_built()


def _check(grid, items, precision, taus=(math.inf,), gradient=False):
    from paper_2605_18389_amd import Plan
    announce(f"row lines {grid} x{items} {precision}")
    G = O.HealpixGrid(grid[1], grid[2]) if grid[0] == "hp" else O.make_grid(*grid)
    rng = np.random.default_rng(items)
    p, q = (0.5 + rng.random((items,) + tuple(G.field_shape)) for _ in range(2))
    tol = 1e-5 if precision == "fp32" else 1e-12
    P = Plan([grid], precision=precision, legendre="recurrence")
    pd, qd = to_dev(p, P.dtype), to_dev(q, P.dtype)
    pick = sorted({0, items // 2, items - 1})
    for tr in (False, True) if taus else (False,):
        out = to_np(P.heat_apply(pd, 1e-3, transpose=tr)).reshape(p.shape)[pick]
        assert rel_l2(out, O.heat_apply(p[pick], G, 1e-3, transpose=tr)) < tol
    for tau in taus:
        phi, psi, info = P.sinkhorn(pd, qd, 0.5, tau, T=3, C=2)
        r = O.sinkhorn(p[pick], q[pick], G, 0.5, tau, T=3, C=2)
        assert rel_l2(to_np(phi).reshape(p.shape)[pick], r["phi"]) < 10 * tol
        assert rel_l2(to_np(psi).reshape(p.shape)[pick], r["psi"]) < 10 * tol
        assert all(info[i]["status"] == 0 for i in pick)
        if gradient:  # a batch against its last pair's own call
            g = to_np(P.divergence_grad(pd, qd, 0.5, T=3, tau=tau)[1]).reshape(p.shape)
            one = to_np(P.divergence_grad(to_dev(p[-1], P.dtype), to_dev(q[-1], P.dtype), 0.5, T=3, tau=tau)[1])
            assert rel_l2(g[-1], one.reshape(p[-1].shape)) < 20 * tol


@pytest.mark.parametrize("precision", ["fp32", "fp64"])
@pytest.mark.parametrize("nlon", [1440, 1458, 1500, 1536, 1599, 1600, 1602, 1620, 2000, 2048])
def test_long_rows(nlon, precision):
    """Lengths whose float64 buffers fit a compute unit's LDS twice or once, of radix 8, 4, 2 and 3 first."""
    _check(("gl", 7, nlon, 7), 2, precision, gradient=True)


@pytest.mark.parametrize("grid,items", [(("gl", 32, 64, 31), 1), (("gl", 32, 64, 31), 56), (("gl", 32, 64, 31), 57),
                                        (("gl", 50, 128, 30), 15), (("gl", 50, 128, 30), 16), (("gl", 50, 256, 30), 15),
                                        (("gl", 50, 256, 30), 16), (("gl", 60, 512, 30), 29), (("gl", 60, 512, 30), 30),
                                        (("gl", 64, 1024, 30), 32), (("gl", 40, 240, 30), 31),
                                        (("gl", 40, 240, 30), 32)])
def test_float64_powers(grid, items):
    """Balanced and unbalanced float64 steps below and from the pair count from which they share a form."""
    _check(grid, items, "fp64", taus=(math.inf, 1.0), gradient=True)


@pytest.mark.parametrize("precision", ["fp32", "fp64"])
@pytest.mark.parametrize("grid,items", [(("gl", 40, 126, 30), 3), (("gl", 40, 132, 30), 1), (("gl", 40, 132, 30), 31),
                                        (("gl", 40, 132, 30), 32), (("gl", 39, 154, 30), 40), (("gl", 39, 182, 30), 39),
                                        (("gl", 20, 198, 20), 2), (("gl", 40, 252, 30), 25), (("gl", 40, 252, 30), 40)])
def test_prime_radices(grid, items, precision):
    """Rows with a radix of 7, 11 or 13 below and from the pair counts (640 and 800) of one wave a pair, balanced and
    unbalanced: in float32 the halves below run on the workgroup kernel, the transforms on 256 lanes."""
    _check(grid, items, precision, taus=(math.inf, 1.0), gradient=True)


def test_balanced_and_unbalanced_on_one_plan():
    """A recorded solve is replayed for calls of its own kind only: the same bits as on a plan of its own."""
    import torch
    from paper_2605_18389_amd import Plan
    announce("balanced and unbalanced on one plan")
    grid = ("gl", 20, 512, 20)
    rng = np.random.default_rng(3)
    one = Plan([grid], precision="fp64", legendre="recurrence")
    p, q = (to_dev(0.5 + rng.random((20, 512)), one.dtype) for _ in range(2))
    for tau in (math.inf, 1.0, math.inf, 10.0):
        own = Plan([grid], precision="fp64", legendre="recurrence")
        a, b = one.sinkhorn(p, q, 0.5, tau, T=5), own.sinkhorn(p, q, 0.5, tau, T=5)
        assert torch.equal(a[0], b[0]) and torch.equal(a[1], b[1]) and a[2] == b[2]


@pytest.mark.parametrize("grid,items,precision", [(("hp", 40, 40), 14, "fp32"), (("hp", 40, 40), 15, "fp32"),
                                                  (("hp", 64, 60), 10, "fp64"), (("hp", 401, 20), 1, "fp32"),
                                                  (("hp", 401, 20), 2, "fp32"), (("hp", 487, 20), 2, "fp32"),
                                                  (("hp", 487, 20), 1, "fp64")])
def test_rings(grid, items, precision):
    """HEALPix below and from the pair count of whole waves a pair, and belts of long primes in both kernels (heat
    applies alone: the oracle takes seconds an apply there)."""
    _check(grid, items, precision, taus=(math.inf, 1.0) if grid[1] < 100 else ())
