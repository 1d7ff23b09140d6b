"""Float32 errors against the float64 plan on the same inputs, over enough inputs that a launch's rounding luck
averages out.  u = 2^-24 is the unit roundoff of float32."""

import numpy as np
import pytest

from helpers import announce, ensure_built

pytestmark = pytest.mark.gpu

U = 2.0 ** -24


@pytest.fixture(scope="module", autouse=True)
def _built():
    ensure_built()


def _plans(grid):
    from paper_2605_18389_amd import Plan
    return (Plan([grid], precision=p, legendre="recurrence") for p in ("fp32", "fp64"))


def _field(P, seed):
    """A float32 field around a mean anywhere in a binade, so that sums of any mantissa are met."""
    import torch
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    mean = 2.0 ** torch.rand(1, dtype=torch.float64, device="cuda", generator=g)
    return (mean * (0.5 + torch.rand(P.field_size(0), dtype=torch.float64, device="cuda", generator=g))).float()


def _rms(x):
    return float(np.sqrt(np.mean(np.square(x))))


@pytest.mark.parametrize("grid", [("gl", 200, 400, 200), ("gl", 256, 512, 256), ("gl", 512, 1024, 512),
                                  ("cc", 721, 1440, 720)])
def test_mean_of_one_field(grid):
    """f_00 of one item (row-split kernel): float64 lane sums, a float32 tree over the lanes, one rounding of the
    result.  A rounding of a mantissa anywhere in its binade is off by 0.425 u rms; the tree's levels carry half
    the weight each, which makes sqrt(2) of that: 0.60 u, and 10 % for 64 samples.  A second rounding of the
    result (0.425 u more, in quadrature: 0.74 u) is over it."""
    announce(f"mean of one field {grid}")
    P, D = _plans(grid)
    e = []
    for seed in range(64):
        x = _field(P, seed)
        c, d = complex(P.analysis(x)[0]), complex(D.analysis(x.double())[0])
        e.append(abs(c - d) / abs(d))
    assert _rms(e) < 0.66 * U, _rms(e) / U


def _workload(**case):
    """Inputs of perf/cases.py's kind."""
    import importlib.util
    import os
    path = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "perf", "cases.py")
    spec = importlib.util.spec_from_file_location("workload_cases", path)
    m = importlib.util.module_from_spec(spec)
    spec.loader.exec_module(m)
    c = dict(ib=0, transpose=False, T=0, tol=0.0, precision="fp32", legendre="recurrence", **case)
    return lambda seed: m.Inputs(c, seed)


def test_unbalanced_gradient():
    """The reverse step undoes u -> u^lam with the exponent 1/lam of the same rounded lam.  With an exponent rounded
    on its own each of the 80 half steps would scale the field by 1 + O(u |log u|), all in one direction: 1.3e-5
    against 8.1e-6 of the row kernel that holds the powers (rms of 12 inputs); the bound lies between."""
    announce("unbalanced gradient")
    P, D = _plans(("hp", 64, 128))
    inputs = _workload(op="attribution", grids="hp 64 128", items="2", t="0.01 0.01", tau="10", field="bumps")
    e = []
    for seed in range(100, 112):
        x = inputs(seed)
        g = P.divergence_grad(x.p, x.q, 4 * x.t, T=40, tau=x.tau)[1].double()
        d = D.divergence_grad(x.p.double(), x.q.double(), 4 * x.t, T=40, tau=x.tau)[1]
        e.append(float((g - d).norm() / d.norm()))
    assert _rms(e) < 1.05e-5, _rms(e)


@pytest.mark.parametrize("grid", [("gl", 90, 180, 90), ("gl", 112, 225, 109), ("gl", 123, 250, 123)])
def test_constant_mode_of_a_batch(grid):
    """A heat apply that leaves the constant mode alone (t = 50), in a tuned batch.  The batch kernel's f_00 is a
    float64 sum, and its rows run on sqrt(4 pi) P, whose degree 0 is 1: the field is b_00, rounded once, 0.29 ulp rms;
    the forward rows' errors, averaged over the latitudes, add 0.05 in quadrature.  With a degree 0 of 1 / sqrt(4 pi)
    the product rounds as well: 0.41 ulp.  512 fields tell 0.35 from either."""
    announce(f"constant mode of a batch {grid}")
    import torch
    P, D = _plans(grid)
    P.set_tuning(0, 8, 0)
    fs, e = P.field_size(0), []
    for k in range(64):
        x = torch.cat([_field(P, 8 * k + i) for i in range(8)])
        out = P.heat_apply(x, 50.0).double().reshape(8, fs)[:, 0]
        ref = D.heat_apply(x.double(), 50.0).reshape(8, fs)[:, 0]
        e += ((out - ref) / 2.0 ** (torch.floor(torch.log2(ref)) - 23)).tolist()
    assert _rms(e) < 0.35, _rms(e)


@pytest.mark.parametrize("grid,items", [(("gl", 130, 260, 130), 2), (("gl", 200, 400, 200), 2),
                                        (("gl", 400, 800, 400), 1), (("cc", 721, 1440, 720), 1)])
def test_constant_mode_of_few_fields(grid, items):
    """As above for the row-split kernel's two-pass form: its rows, b and synthesis sums are
    float64, so with f_00 summed in float64 the constant mode is rounded once, on its way out.  A float32 tree over
    the lanes adds roundings of 0.425 u each, half the weight a level up: 0.29 and 0.45 in quadrature, 0.5 ulp."""
    announce(f"constant mode of few fields {grid} x{items}")
    import torch
    P, D = _plans(grid)
    fs, e = P.field_size(0), []
    for k in range(192 // items):
        x = torch.cat([_field(P, items * k + i) for i in range(items)])
        out = P.heat_apply(x, 50.0).double().reshape(items, fs)[:, 0]
        ref = D.heat_apply(x.double(), 50.0).reshape(items, fs)[:, 0]
        e += ((out - ref) / 2.0 ** (torch.floor(torch.log2(ref)) - 23)).tolist()
    assert _rms(e) < 0.36, _rms(e)


@pytest.mark.parametrize("nside", [251, 401, 509])
def test_rings_of_long_primes(nside):
    """Coefficients beyond the mean on grids whose belt is rings of 4p pixels, p prime: the radix-p stage sums
    (p - 1) / 2 products.  The rounding of a running sum of n terms grows as sqrt(n / 2), in sums of
    32 as sqrt(16 + n / 64): 11.3 against 4.5 at p = 509.  The bounds are 1.25 times the errors of the Bluestein
    transform that row_kernel runs on these rings (7.9e-7, 1.07e-6 and 1.23e-6, rms of 12 inputs)."""
    announce(f"rings of long primes {nside}")
    P, D = _plans(("hp", nside, 400))
    e = []
    for seed in range(12):
        x = _field(P, seed)
        c, d = P.analysis(x)[1:].to(dtype=D.analysis(x.double()).dtype), D.analysis(x.double())[1:]
        e.append(float((c - d).norm() / d.norm()))
    assert _rms(e) < 1.25 * {251: 7.9e-7, 401: 1.07e-6, 509: 1.23e-6}[nside], _rms(e)


@pytest.mark.parametrize("nlon", [64, 128, 256, 512, 1024])
def test_divide_by_large_kernel_values(nlon):
    """Marginals of a scale that takes the gauge times K v to 1.5e38, above 2^126, whose reciprocal is subnormal,
    while every scaling stays a normal number.  As the float64 solve, to the transforms' rounding: a few u in each
    of the four halves."""
    announce(f"divide by large kernel values {nlon}")
    P, D = _plans(("gl", 1024 * 64 // nlon, nlon, 8))
    p, q = ((x / x.mean() * (1.5e38 / P.field_size(0))).float() for x in (_field(P, k).double() for k in (1, 2)))
    # u-hat_1 = p, its sum g = 1.5e38, v-hat_1 = q / p, and u-hat_2 = p / (g K v-hat_1)
    phi, psi, info = P.sinkhorn(p, q, 4.0, T=2)
    dphi, dpsi, dinfo = D.sinkhorn(p.double(), q.double(), 4.0, T=2)
    assert info[0]["breakdown_iter"] == 0 and dinfo[0]["breakdown_iter"] == 0
    assert float((phi.double() - dphi).norm() / dphi.norm()) < 20 * U
    assert float((psi.double() - dpsi).norm() / dpsi.norm()) < 20 * U
