"""Plans of different sizes used from host threads of their own: kernels of one instantiation with different amounts
of LDS, each thread's results against the oracle."""

import threading

import numpy as np
import pytest

import oracle as O

from helpers import announce, ensure_built, rel_l2, to_dev, to_np

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _built():
    ensure_built()


@pytest.mark.parametrize("precision,legendre", [("fp64", "recurrence"), ("fp64", "table"), ("fp32", "table")])
def test_plans_on_threads(precision, legendre):
    import torch
    from paper_2605_18389_amd import Plan
    announce(f"plans on threads {precision} {legendre}")
    grids = [("gl", 300, 2048, 60), ("gl", 380, 1620, 40), ("gl", 440, 1728, 50), ("gl", 6, 2000, 6)]
    tol = 1e-12 if precision == "fp64" else 1e-5
    errs, fails = [None] * len(grids), []

    def work(i):
        try:
            grid = grids[i]
            G = O.make_grid(*grid)
            v = 0.5 + np.random.default_rng(i).random((3, grid[1], grid[2]))
            with torch.cuda.stream(torch.cuda.Stream()):
                P = Plan([grid], precision=precision, legendre=legendre)
                x = to_dev(v, P.dtype)
                out = [to_np(P.heat_apply(x, 1e-3)) for _ in range(5)][-1].reshape(v.shape)
            errs[i] = rel_l2(out, O.heat_apply(v, G, 1e-3))
        except Exception as e:  # reported by the test's thread
            fails.append(repr(e))

    threads = [threading.Thread(target=work, args=(i,)) for i in range(len(grids))]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not fails and max(errs) < tol, (fails, errs)
