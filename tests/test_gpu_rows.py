"""Row transforms against the oracle at the edges of their launch shapes: compile-time lengths with one and
with many row pairs (whole, half and quarter waves per pair), run-time lengths (large primes, odd lengths, the
shortest and longest rows), groups that a grid's rows do not fill, the equator row of odd grids, HEALPix rings of
prime sizes, and the adjoint's row steps of a batch against the same items run one at a time."""

import math

import numpy as np
import pytest

import oracle as O

from helpers import announce, ensure_built, rel_l2, to_dev, to_np

pytestmark = pytest.mark.gpu

# (grid, items): see row_wave_shape for the lines between the shapes
SHAPES = [
    (("gl", 31, 64, 31), 1), (("gl", 33, 64, 20), 5), (("cc", 65, 128, 64), 3), (("gl", 37, 256, 37), 2),
    (("gl", 21, 512, 20), 3), (("gl", 16, 1024, 16), 2), (("gl", 17, 1024, 16), 120),
    (("gl", 45, 180, 44), 48), (("gl", 45, 180, 20), 720), (("gl", 32, 360, 30), 70), (("gl", 31, 360, 20), 520),
    (("gl", 19, 720, 19), 110), (("gl", 8, 6, 3), 1), (("gl", 9, 14, 7), 3), (("gl", 40, 66, 33), 40),
    (("gl", 41, 202, 30), 2), (("gl", 40, 150, 40), 30), (("gl", 12, 1200, 12), 3), (("gl", 6, 2047, 6), 2),
    (("gl", 5, 2048, 5), 2), (("gl", 5, 1999, 5), 1), (("hp", 1, 2), 1), (("hp", 17, 34), 2), (("hp", 61, 90), 9),
    (("hp", 67, 90), 1), (("hp", 127, 40), 1),
]


@pytest.fixture(scope="module", autouse=True)
def _built():
    ensure_built()


def _oracle_grid(g):
    return O.HealpixGrid(g[1], g[2]) if g[0] == "hp" else O.make_grid(*g)


def _fields(G, n, seed):
    return 0.5 + np.random.default_rng(seed).random((n,) + tuple(G.field_shape))


@pytest.mark.parametrize("precision,tol", [("fp32", 1e-5), ("fp64", 1e-12)])
@pytest.mark.parametrize("grid,items", SHAPES)
def test_heat_apply_row_shapes(grid, items, precision, tol):
    from paper_2605_18389_amd import Plan
    announce(f"rows {grid} x{items} {precision}")
    G = _oracle_grid(grid)
    v = _fields(G, items, 1)
    P = Plan([grid], precision=precision, legendre="recurrence")
    t = 1e-3
    for tr in (False, True):
        out = to_np(P.heat_apply(to_dev(v, P.dtype), t, transpose=tr)).reshape(v.shape)
        pick = sorted({0, items // 2, items - 1})
        ref = O.heat_apply(v[pick], G, t, transpose=tr)
        assert rel_l2(out[pick], ref) < tol
        # every item of a batch equals the item alone, up to the two launches' rounding
        one = to_np(P.heat_apply(to_dev(v[items - 1], P.dtype), t, transpose=tr)).reshape(v[0].shape)
        assert rel_l2(out[items - 1], one) < tol


@pytest.mark.parametrize("precision,tol", [("fp32", 1e-4), ("fp64", 1e-10)])
@pytest.mark.parametrize("tau", [math.inf, 1.0])
@pytest.mark.parametrize("grid,items", [(("gl", 33, 64, 20), 5), (("gl", 17, 1024, 16), 120), (("gl", 45, 180, 44), 48),
                                        (("gl", 31, 360, 20), 520), (("gl", 19, 720, 19), 110),
                                        (("gl", 41, 202, 30), 2), (("gl", 12, 1200, 12), 3), (("hp", 17, 34), 2)])
def test_sinkhorn_row_shapes(grid, items, tau, precision, tol):
    from paper_2605_18389_amd import Plan
    announce(f"sinkhorn rows {grid} x{items} tau={tau} {precision}")
    G = _oracle_grid(grid)
    p, q = _fields(G, items, 2), _fields(G, items, 3)
    P = Plan([grid], precision=precision, legendre="recurrence")
    phi, psi, info = P.sinkhorn(to_dev(p, P.dtype), to_dev(q, P.dtype), 0.5, tau, T=4, C=2)
    pick = sorted({0, items // 2, items - 1})
    r = O.sinkhorn(p[pick], q[pick], G, 0.5, tau, T=4, C=2)
    assert rel_l2(to_np(phi).reshape(p.shape)[pick], r["phi"]) < tol
    assert rel_l2(to_np(psi).reshape(p.shape)[pick], r["psi"]) < tol
    for k, i in enumerate(pick):
        assert info[i]["status"] == 0
        assert abs(info[i]["cost"] - r["cost"][k]) <= tol * abs(r["cost"][k])
        assert abs(info[i]["err"] - r["err"][k]) <= 10 * tol
        assert abs(info[i]["kratio"] - r["kratio"][k]) <= 10 * tol


@pytest.mark.parametrize("precision,tol", [("fp32", 2e-4), ("fp64", 1e-9)])
@pytest.mark.parametrize("tau", [math.inf, 1.0])
@pytest.mark.parametrize("grid,pairs", [(("gl", 45, 180, 44), 26), (("gl", 31, 360, 20), 40), (("gl", 19, 720, 19), 60),
                                        (("gl", 33, 64, 20), 3), (("gl", 41, 202, 30), 2), (("hp", 17, 34), 3)])
def test_gradient_row_shapes(grid, pairs, tau, precision, tol):
    """A batch's gradient (wave-per-pair rows) against each pair's own call, and one pair's directional
    derivative against the oracle's central differences."""
    from paper_2605_18389_amd import Plan, synth
    announce(f"gradient rows {grid} x{pairs} tau={tau} {precision}")
    G = _oracle_grid(grid)
    p, q = _fields(G, pairs, 4), _fields(G, pairs, 5)
    P = Plan([grid], precision=precision, legendre="recurrence")
    S, g, _ = P.divergence_grad(to_dev(p, P.dtype), to_dev(q, P.dtype), 0.5, T=4, tau=tau)
    g = to_np(g).reshape(p.shape)
    i = pairs - 1
    S1, g1, _ = P.divergence_grad(to_dev(p[i], P.dtype), to_dev(q[i], P.dtype), 0.5, T=4, tau=tau)
    assert rel_l2(g[i], to_np(g1).reshape(p[i].shape)) < tol
    if precision == "fp64":
        d = synth.mass_preserving_directions(6, p[i], G.area, 1)
        fd = float(O.fd_directional(p[i], q[i], d, G, 0.5, 4, h=1e-4, tau=tau)[0])
        scale = float(np.linalg.norm(g[i])) * float(np.linalg.norm(d[0]))
        assert abs(float((g[i] * d[0]).sum()) - fd) <= 1e-6 * scale
