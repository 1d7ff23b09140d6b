"""Per-call data of a heat apply: item counts around the launch-argument sizes (2, 32, 96 items) with a heat time
each, over two grids; calls queued behind one another without a wait; a call under stream capture stays refused."""

import numpy as np
import pytest

import oracle as O

from helpers import announce, ensure_built, rel_l2, to_dev, to_np

pytestmark = pytest.mark.gpu

GRIDS = [("gl", 8, 16, 8), ("gl", 12, 20, 10)]


@pytest.fixture(scope="module", autouse=True)
def _built():
    ensure_built()


@pytest.mark.parametrize("precision,tol", [("fp32", 1e-5), ("fp64", 1e-12)])
@pytest.mark.parametrize("n", [1, 2, 3, 32, 33, 96, 97])
def test_items_of_a_call(n, precision, tol):
    from paper_2605_18389_amd import Plan
    announce(f"items of a call {n} {precision}")
    rng = np.random.default_rng(n)
    goi = [int(k) for k in rng.integers(0, 2, n)]
    gs = [O.make_grid(*g) for g in GRIDS]
    t = 10.0 ** rng.uniform(-4, -1, n)
    fields = [0.5 + rng.random((gs[k].nlat, gs[k].nlon)) for k in goi]
    P = Plan(GRIDS, precision=precision, legendre="recurrence")
    v = to_dev(np.concatenate([f.ravel() for f in fields]), P.dtype)
    first = P.heat_apply(v, t, grid_of_item=goi)
    second = P.heat_apply(first, t[::-1].copy(), grid_of_item=goi)   # queued behind the first
    outs = to_np(first), to_np(second)
    off = 0
    for i, k in enumerate(goi):
        m = gs[k].nlat * gs[k].nlon
        a = O.heat_apply(fields[i], gs[k], t[i])
        assert rel_l2(outs[0][off:off + m].reshape(a.shape), a) < tol
        b = O.heat_apply(a, gs[k], t[n - 1 - i])
        assert rel_l2(outs[1][off:off + m].reshape(b.shape), b) < 2 * tol
        off += m


def test_call_under_capture_is_refused():
    import torch
    from paper_2605_18389_amd import Plan
    from paper_2605_18389_amd.binding import E_HIP, ShotError
    announce("capture refused")
    P = Plan(GRIDS[:1], precision="fp32", legendre="recurrence")
    v = torch.ones(8, 16, device="cuda")
    ref = P.heat_apply(v, 1e-3)
    torch.cuda.synchronize()
    s = torch.cuda.Stream()
    g = torch.cuda.CUDAGraph()
    code = None
    with torch.cuda.stream(s):
        out = torch.empty_like(v)
        g.capture_begin()
        try:
            P.heat_apply(v, 1e-3, out=out)
        except ShotError as e:
            code = e.code
        g.capture_end()
    torch.cuda.synchronize()
    assert code == E_HIP
    assert torch.equal(P.heat_apply(v, 1e-3), ref)
