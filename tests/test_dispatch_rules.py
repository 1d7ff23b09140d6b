"""Host rules that choose a kernel, called in the built library (CPU)."""

import ctypes
import os

import pytest


@pytest.fixture(scope="module")
def lib():
    from paper_2605_18389_amd import binding
    if not os.path.exists(binding.LIB_PATH):
        from paper_2605_18389_amd.build import build
        build()
    binding._torch()
    return ctypes.CDLL(binding.LIB_PATH)


# (mode, items, latitude pairs, float64, row-split by two) and which kernel measured faster there
TIMED = [(2, 5, 180, 0, 1, 0), (2, 8, 180, 1, 0, 0), (2, 12, 180, 0, 1, 0), (2, 16, 180, 0, 1, 1), (2, 17, 193, 0, 1, 0),
         (2, 24, 193, 0, 1, 1), (2, 8, 193, 0, 1, 1), (2, 5, 361, 0, 0, 0), (2, 6, 361, 0, 0, 1), (2, 10, 361, 0, 0, 0),
         (2, 12, 91, 0, 1, 0), (2, 17, 91, 0, 1, 1), (2, 64, 17, 0, 1, 1), (1, 5, 180, 0, 1, 0), (1, 8, 180, 0, 1, 1),
         (1, 12, 260, 0, 1, 0), (1, 16, 260, 0, 1, 1), (1, 12, 180, 0, 1, 1), (1, 5, 361, 0, 0, 0), (1, 12, 361, 0, 0, 1),
         (2, 12, 180, 1, 0, 1), (2, 12, 150, 1, 1, 0), (1, 18, 200, 0, 1, 0), (1, 18, 200, 1, 0, 1),
         (0, 5, 260, 0, 1, 0), (0, 5, 260, 1, 0, 0), (0, 8, 260, 0, 1, 1), (0, 5, 181, 0, 1, 1), (0, 8, 361, 0, 0, 1)]


@pytest.mark.parametrize("mode,items,h,f64,pairs,batch", TIMED)
def test_batch_kernel_line(lib, mode, items, h, f64, pairs, batch):
    f = lib._ZN4shot12batch64_paysEiiibb
    f.argtypes = [ctypes.c_int] * 3 + [ctypes.c_bool] * 2
    f.restype = ctypes.c_bool
    assert f(mode, items, (h + 63) // 64, bool(f64), bool(pairs)) == bool(batch)


def test_limits_of_the_float64_kernels(lib):
    """The sizes that include/shot.h states: tables of 896 rows; recurrence batches of 640 rows, or 768 up to L = 800."""
    t, r = lib._ZN4shot8t64_fitsEi, lib._ZN4shot8r64_fitsEii
    t.argtypes, r.argtypes = [ctypes.c_int], [ctypes.c_int] * 2
    t.restype = r.restype = ctypes.c_bool
    assert [h for h in range(1, 1025) if t(h)] == list(range(1, 449))
    assert all(r(1024, h) for h in range(1, 321))
    assert all(r(800, h) and not r(801, h) for h in range(321, 385))
    assert not any(r(1, h) for h in range(385, 1025))
    text = open(os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "include", "shot.h")).read()
    text = " ".join(text.replace("*", " ").split())
    assert "float64 tables of at most 896 rows" in text and "at most 640 rows, or 768 with L <= 800" in text
