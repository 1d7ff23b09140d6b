"""Calls on a stream under capture are refused before any launch, the no-allocation heat apply among them, whatever
their item count; the capture stays valid, and the plan works afterwards."""

import ctypes
import os

import numpy as np
import pytest

from helpers import announce, ensure_built

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _built():
    ensure_built()


@pytest.mark.parametrize("items", [1, 33, 97])
@pytest.mark.parametrize("name", ["shot_heat_apply_noalloc", "shot_heat_apply"])
def test_capture_is_refused(name, items):
    import torch
    from paper_2605_18389_amd import Plan
    from paper_2605_18389_amd.binding import E_HIP, OK
    announce(f"capture {name} x{items}")
    P = Plan([("gl", 8, 16, 8)], precision="fp32", legendre="recurrence")
    v = torch.rand(items, 8, 16, device="cuda") + 0.5
    ref = P.heat_apply(v, 1e-3)
    out, kept = torch.zeros_like(v), torch.zeros(4, device="cuda")
    t = np.full(items, 1e-3)
    goi = (ctypes.c_int32 * items)()

    def call():
        return getattr(P.lib, name)(P.handle, goi, items, t.ctypes.data_as(ctypes.POINTER(ctypes.c_double)),
                                    ctypes.c_void_p(v.data_ptr()), ctypes.c_void_p(out.data_ptr()), 0,
                                    ctypes.c_void_p(torch.cuda.current_stream().cuda_stream))

    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.stream(torch.cuda.Stream()):
        graph.capture_begin()
        kept += 1
        code = call()
        graph.capture_end()
    assert code == E_HIP
    for k in (1, 2):
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(kept, torch.full_like(kept, k)) and not out.any()
    assert call() == OK
    torch.cuda.synchronize()
    assert torch.equal(out, ref)


def test_header_does_not_offer_capture():
    path = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "include", "shot.h")
    assert "code under\n * HIP graph capture" not in open(path).read()
