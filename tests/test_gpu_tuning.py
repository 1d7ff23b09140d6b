"""Autotuning reports what runs: a float32 table of up to 1024 rows has one matrix-core form, so that no tile count
but the smallest can be picked; a count that was set by hand is accepted and changes nothing."""

import numpy as np
import pytest

import oracle as O

from helpers import announce, ensure_built, rel_l2, to_dev, to_np

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _built():
    ensure_built()


def test_table_tile_counts():
    import torch
    from paper_2605_18389_amd import Plan
    announce("table tile counts")
    picked = set()
    for nlat in (32, 64, 96, 128, 160, 192):
        P = Plan([("gl", nlat, 2 * nlat, nlat)], precision="fp32", legendre="table")
        P.autotune(0, 40)
        picked.add(P.get_tuning(0))
    assert picked <= {(0, 1)} | {(ib, -1) for ib in (1, 2, 4, 8)}, picked
    grid = ("gl", 40, 80, 40)
    G = O.make_grid(*grid)
    v = 0.5 + np.random.default_rng(1).random((17, 40, 80))
    P = Plan([grid], precision="fp32", legendre="table")
    outs = []
    for nt in (0, 1, 2, 4):
        P.set_tuning(0, 0, nt)
        outs.append(P.heat_apply(to_dev(v, P.dtype), 1e-3))
    assert all(torch.equal(outs[0], o) for o in outs[1:])
    assert rel_l2(to_np(outs[0]).reshape(v.shape), O.heat_apply(v, G, 1e-3)) < 1e-5
