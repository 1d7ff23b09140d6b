"""Workloads of the library for timing: heat smoothing, transforms, Sinkhorn
solves, divergences and their gradients, through the package's public entry
points.

A case is a dict of plain values:

  op        smooth (Plan.heat_apply), analysis, synthesis, solve (Plan.sinkhorn),
            divergence, gradient (Plan.divergence_grad) or attribution
            (Plan.divergence_grad and Plan.regional_rms)
  grids     grids of the plan, e.g. "cc 721 1440 720" (kind, rows, columns, band
            limit) or "hp 64 128" (Nside, band limit), separated by ";"
  items     items (pairs) on each grid, separated by ";"
  precision, legendre
            as Plan takes them
  ib        items per workgroup the program's plan is tuned to (0: automatic)
  transpose smooth: the transpose of the operator
  t         smallest and largest heat time "a b" (log-spaced over the items)
  T, tol, tau
            iterations, tolerance and marginal penalty (0: balanced; "mixed":
            every other pair unbalanced, tau in {0.1, 1, 10}, masses 1 and 1.05)
  field     temperature, bumps (small anomalies of a smooth density), contrast
            (large ones) or uniform

Scalars of a float32 plan carry float32 accuracy and are returned as such.  The
divergence of a balanced pair is the difference of its three costs, often a
thousand times smaller than they are: the costs themselves are returned there.
"""

import math

import numpy as np
import torch

DEV = "cuda"
REGIONS = {"tropics": (-23.5, 23.5), "itcz": (-10.0, 10.0), "nh_midlatitudes": (30.0, 60.0),
           "sh_midlatitudes": (-60.0, -30.0), "arctic": (66.5, 90.5)}


def _case(op, grids, items, precision="fp32", legendre="recurrence", **more):
    c = {"op": op, "grids": grids, "items": items, "precision": precision, "legendre": legendre, "ib": 0,
         "transpose": False, "t": "0.01 0.01", "T": 0, "tol": 0.0, "tau": "0", "field": "temperature"}
    c.update(more)
    return c


def listed():
    return [
        # the smallest calls: one vMF-like field smoothed at eight heat times (the
        # heat-against-matrix study's batch), float64, the plan's default Legendre mode
        _case("smooth", "cc 33 64 32", "8", "fp64", "auto", t="0.00025 2.5", field="bumps", name="smooth_cc33_x8_fp64"),
        # one quarter-degree field smoothed in float32: the serving call
        _case("smooth", "cc 721 1440 720", "1", t="0.0001 0.0001", name="smooth_cc721"),
        # an ensemble of half-degree fields with the plan's defaults (a float32 table)
        _case("smooth", "gl 360 720 360", "16", legendre="auto", t="0.001 0.01", name="smooth_gl360_x16_table"),
        # a batch of one-degree fields in split bfloat16
        _case("smooth", "gl 180 360 180", "24", "bf16x3", t="0.001 0.01", name="smooth_gl180_x24_bf16x3"),
        # spectra of twelve monthly one-degree fields, defaults
        _case("analysis", "gl 180 360 180", "12", legendre="auto", name="analysis_gl180_x12_table"),
        # float64 fields from spectra on a grid of odd row count
        _case("synthesis", "gl 193 400 193", "2", "fp64", name="synthesis_gl193_x2_fp64"),
        # the paper's runtime workload: uniform random fields, eps = 0.1, delta = 1e-9, float64
        _case("solve", "cc 129 256 128", "1", "fp64", t="0.025 0.025", T=100, tol=1e-9, field="uniform",
              name="solve_cc129_fp64"),
        # the quarter-degree solve in float32
        _case("solve", "cc 721 1440 720", "1", T=50, name="solve_cc721"),
        # the same solve with the bfloat16 Legendre table
        _case("solve", "cc 721 1440 720", "1", "bf16", "table", T=50, name="solve_cc721_bf16_table"),
        # uneven batch of balanced and unbalanced pairs over three grids, tuned as a batch program tunes it
        _case("divergence", "gl 90 180 90;gl 180 360 180;gl 360 720 360", "12;12;8", ib=8, t="0.003 0.01", T=30,
              tau="mixed", field="bumps", name="divergence_uneven_x32"),
        # one optimisation step on half-degree pairs: the divergence and its gradient
        _case("gradient", "gl 360 720 360", "8", ib=8, T=40, field="contrast", name="gradient_gl360_x8"),
        # the climate study's step on HEALPix: unbalanced gradients and regional indices
        _case("attribution", "hp 64 128", "8", t="0.0025 0.0025", T=40, tau="1", field="bumps",
              name="attribution_hp64_x8"),
    ]


def _smooth5(n):
    """The next length from n on whose prime factors are 2, 3 and 5."""
    while True:
        k = n
        for p in (2, 3, 5):
            while k % p == 0:
                k //= p
        if k == 1:
            return n
        n += 1


def draw(rng):
    def log_int(a, b):
        return int(round(math.exp(rng.uniform(math.log(a), math.log(b)))))

    def latlon(lmax, lmin=8):
        L = max(lmin, min(lmax, log_int(lmin, lmax)))
        nlon = 2 * L if rng.random() < 0.25 else _smooth5(2 * L)  # rows as given, or padded to a fast length
        kind = rng.choice(("gl", "gl", "cc"))
        nlat = L + (rng.choice((0, 0, 1, 3)) if kind == "gl" else 1)
        return "%s %d %d %d" % (kind, nlat, nlon, L), L

    def count(L, cap):  # cap: items * L^3
        return max(1, min(64, log_int(1, 64), int(cap / L ** 3)))

    op = rng.choice(("smooth", "smooth", "smooth", "analysis", "synthesis", "solve", "solve", "divergence", "gradient",
                     "attribution"))
    if op in ("smooth", "analysis", "synthesis"):
        cap = 16 * 360 ** 3
        precision = rng.choice(("fp64", "fp32", "fp32", "fp32", "bf16x3") if op == "smooth" else ("fp64", "fp32", "fp32"))
        legendre = "recurrence" if precision == "bf16x3" else rng.choice(("auto", "recurrence"))
        if op == "smooth" and rng.random() < 0.2:
            nside = log_int(4, 128)
            return _case(op, "hp %d %d" % (nside, 2 * nside), str(count(2 * nside, cap)),
                         "fp32" if precision == "bf16x3" else precision, legendre, t="0.001 0.1", field="bumps")
        g, L = latlon(720)
        return _case(op, g, str(count(L, cap)), precision, legendre, transpose=op == "smooth" and rng.random() < 0.25,
                     t="%.5f %.5f" % (1.0 / L ** 1.5, 0.05 + 1.0 / L), field=rng.choice(("temperature", "bumps")))
    cap, T = 4e10, rng.choice((20, 30, 50))
    if op == "solve":
        form = rng.randrange(5)
        if form == 0:  # the paper's runtime workload over its resolutions
            L = log_int(16, 256)
            return _case(op, "cc %d %d %d" % (L + 1, 2 * L, L), "1", "fp64", rng.choice(("auto", "recurrence")),
                         t="0.025 0.025", T=100, tol=1e-9, field="uniform")
        if form == 1:
            nside = log_int(16, 128)
            return _case(op, "hp %d %d" % (nside, 2 * nside), "1", rng.choice(("fp32", "fp64")), t="0.025 0.025", T=T,
                         field="uniform")
        if form == 2:
            L = log_int(90, 720)
            return _case(op, "cc %d %d %d" % (L + 1, _smooth5(2 * L), L), "1", "bf16", "table", T=T, field="bumps")
        g, L = latlon(720, 32)
        n = count(L, cap / (2 * T))
        big = n >= 8 and L <= 512
        return _case(op, g, str(n), "fp32", "recurrence" if big else rng.choice(("auto", "recurrence")),
                     ib=8 if big else 0, T=T, field="bumps")
    if op == "divergence":
        gs = [latlon(360, 32) for _ in range(rng.choice((1, 2, 3)))]
        gs.sort(key=lambda x: x[1])
        ns = [count(L, cap / (6 * T * len(gs))) for _, L in gs]
        mixed = rng.random() < 0.5
        return _case(op, ";".join(g for g, _ in gs), ";".join(map(str, ns)), rng.choice(("fp32", "fp32", "fp64")),
                     ib=0 if sum(ns) < 8 else 8, t="0.003 0.01" if mixed else "0.01 0.02", T=T,
                     tau="mixed" if mixed else "0", field="bumps" if mixed else "contrast")
    if op == "gradient":
        g, L = latlon(360, 32)
        n = count(L, cap / (10 * T))
        return _case(op, g, str(n), ib=8 if n >= 3 else 0, T=T, field="contrast")
    nside = log_int(16, 96)
    return _case(op, "hp %d %d" % (nside, 2 * nside), str(min(8, count(2 * nside, cap / (10 * T)))),
                 rng.choice(("fp32", "fp64")), t="0.0025 0.01", T=T, tau="1", field="bumps")


# --------------------------------------------------------------------- grids
class Geometry:
    """Nodes, weights and points of one grid in float64, written from the grids' definitions."""

    def __init__(self, spec):
        f = spec.split()
        self.kind = f[0]
        if self.kind == "hp":
            n, self.L = int(f[1]), int(f[2])
            self.spec = ("hp", n, self.L)
            i = np.arange(1, 4 * n)
            ii = np.minimum(i, 4 * n - i)
            cap = ii < n
            z = np.where(cap, 1.0 - ii * ii / (3.0 * n * n), 4.0 / 3.0 - 2.0 * ii / (3.0 * n))
            self.x = np.where(i <= 2 * n, z, -z)
            self.npix = np.where(cap, 4 * ii, 4 * n)
            self.phi0 = np.where(cap, np.pi / (4.0 * ii), ((ii - n + 1) % 2) * np.pi / (4.0 * n))
            self.nlat, self.nlon = 4 * n - 1, 4 * n
            self.row_area = np.full(self.nlat, 4 * np.pi / (12.0 * n * n))
        else:
            self.nlat, self.nlon, self.L = int(f[1]), int(f[2]), int(f[3])
            self.spec = (self.kind, self.nlat, self.nlon, self.L)
            if self.kind == "gl":
                x, w = np.polynomial.legendre.leggauss(self.nlat)
                self.x, w = x[::-1].copy(), w[::-1].copy()
            else:
                N = self.nlat - 1
                th = np.pi * np.arange(self.nlat) / N
                k = np.arange(1, N // 2 + 1)
                b = np.where(2 * k == N, 1.0, 2.0)
                w = (1.0 - (b / (4.0 * k * k - 1.0) * np.cos(2.0 * np.outer(th, k))).sum(1)) * 2.0 / N
                w[0] /= 2
                w[-1] /= 2
                self.x = np.cos(th)
            self.npix = np.full(self.nlat, self.nlon)
            self.phi0 = np.zeros(self.nlat)
            self.row_area = w * 2 * np.pi / self.nlon
        self.n = int(self.npix.sum())
        dev = lambda a: torch.as_tensor(np.asarray(a, dtype=np.float64), device=DEV)  # noqa: E731
        rep = torch.as_tensor(self.npix, device=DEV)
        start = np.cumsum(self.npix) - self.npix
        k = torch.arange(self.n, device=DEV, dtype=torch.float64) - torch.repeat_interleave(dev(start), rep)
        phi = torch.repeat_interleave(dev(self.phi0), rep) + 2 * math.pi * k / torch.repeat_interleave(
            dev(self.npix), rep)
        z = torch.repeat_interleave(dev(self.x), rep)
        s = torch.sqrt(torch.clamp(1 - z * z, min=0.0))
        self.points = torch.stack([torch.cos(phi) * s, torch.sin(phi) * s, z], -1)
        self.area = torch.repeat_interleave(dev(self.row_area), rep)


_geometry = {}


def _geom(spec):
    if spec not in _geometry:
        if len(_geometry) > 8:
            _geometry.clear()
        _geometry[spec] = Geometry(spec)
    return _geometry[spec]


def _bumps(g, gen, kap, amp):
    """Sum of 8 bumps amp e^{kappa (mu . x - 1)} with random centres, kappa and amp in the given ranges."""
    mu = torch.randn(8, 3, dtype=torch.float64, device=DEV, generator=gen)
    mu = mu / mu.norm(dim=1, keepdim=True)
    r = torch.rand(2, 8, dtype=torch.float64, device=DEV, generator=gen)
    k, a = kap[0] + (kap[1] - kap[0]) * r[0], amp[0] + (amp[1] - amp[0]) * r[1]
    b = torch.zeros_like(g.area)
    for j in range(8):
        b += a[j] * torch.exp(k[j] * (g.points @ mu[j] - 1))
    return b


def _fields(g, kind, n, gen, mass, climate):
    """n densities on grid g, float64, [n, points]; `climate` is what the fields of a call have in common."""
    out = []
    for i in range(n):
        if kind == "uniform":
            f = torch.rand(g.n, dtype=torch.float64, device=DEV, generator=gen)
        elif kind == "temperature":  # zonal background with warm and cold anomalies
            b = _bumps(g, gen, (5.0, 50.0), (-0.2, 0.2))
            f = torch.clamp((1 - g.points[:, 2] ** 2) * (1 + b), min=0.0) + 1e-3
        else:                        # anomalies of a smooth climatology bounded below
            a = 0.25 if kind == "contrast" else 0.05
            f = climate + _bumps(g, gen, (3.0, 15.0), (-a, a))
        out.append(f * (mass[i] / (g.area * f).sum()))
    return torch.stack(out)


class Inputs:
    """A case's host parameters and device inputs, from the seed alone."""

    def __init__(self, case, seed):
        self.geoms = [_geom(s) for s in case["grids"].split(";")]
        self.counts = [int(k) for k in case["items"].split(";")]
        self.goi = sum(([g] * k for g, k in enumerate(self.counts)), [])
        n = len(self.goi)
        self.dtype = torch.float64 if case["precision"] == "fp64" else torch.float32
        lo, hi = (float(x) for x in case["t"].split())
        self.t = np.exp(np.linspace(math.log(lo), math.log(hi), n)) if n > 1 else np.array([lo])
        if case["tau"] == "mixed":
            self.tau = np.array([math.inf if i % 2 == 0 else (0.1, 1.0, 10.0)[(i // 2) % 3] for i in range(n)])
        else:
            self.tau = np.full(n, float(case["tau"]) or math.inf)
        gen = torch.Generator(device=DEV)
        gen.manual_seed(int(seed))
        pair = case["op"] in ("solve", "divergence", "gradient", "attribution")
        p, q, i = [], [], 0
        for g, k in zip(self.geoms, self.counts):
            qm = [1.0 if math.isinf(x) else 1.05 for x in self.tau[i:i + k]]
            i += k
            if case["op"] == "synthesis":
                L = g.L  # spectra of decaying power; order 0 is real
                m = torch.arange(L, device=DEV)
                l_of = torch.cat([torch.arange(j, L, device=DEV) for j in range(L)])
                m_of = torch.repeat_interleave(m, L - m)
                c = torch.randn(k, l_of.numel(), 2, dtype=torch.float64, device=DEV, generator=gen)
                c = c / (1.0 + l_of.double())[:, None]
                c[:, m_of == 0, 1] = 0.0
                p.append(c.reshape(-1))
                continue
            climate = 1.0 + _bumps(g, gen, (3.0, 15.0), (0.1, 0.5))
            p.append(_fields(g, case["field"], k, gen, [1.0] * k, climate).reshape(-1))
            if pair:
                q.append(_fields(g, case["field"], k, gen, qm, climate).reshape(-1))
        self.p = torch.cat(p).to(self.dtype)
        self.q = torch.cat(q).to(self.dtype) if q else None


_plan = {}


def _plan_of(case, geoms):
    """The program's plan: made once and kept for all its inputs (the last configuration's is kept)."""
    from paper_2605_18389_amd import Plan
    key = (case["grids"], case["precision"], case["legendre"], case["ib"])
    if key not in _plan:
        _plan.clear()
        P = Plan([g.spec for g in geoms], precision=case["precision"], legendre=case["legendre"])
        for k in range(len(geoms)):
            if case["ib"]:
                P.set_tuning(k, case["ib"], 0)
        _plan[key] = P
    return _plan[key]


def prepare(case, seed):
    x = Inputs(case, seed)
    return {"case": case, "x": x, "plan": _plan_of(case, x.geoms)}


def _scalars(x, values):
    return np.asarray(values, dtype=np.float64 if x.dtype == torch.float64 else np.float32)


def run(state):
    case, x, P = state["case"], state["x"], state["plan"]
    op = case["op"]
    goi = x.goi if len(x.geoms) > 1 else None
    eps = 4.0 * x.t
    if op == "smooth":
        return P.heat_apply(x.p, x.t, grid_of_item=goi, transpose=case["transpose"])
    if op == "analysis":
        return P.analysis(x.p, grid_of_item=goi)
    if op == "synthesis":
        return P.synthesis(x.p, grid_of_item=goi)
    if op == "solve":
        phi, psi, info = P.sinkhorn(x.p, x.q, eps, x.tau, T=case["T"], tol=case["tol"], grid_of_item=goi)
        return {"phi": phi, "psi": psi, "cost": _scalars(x, [i["cost"] for i in info]), "iters": info[0]["iters"]}
    if op == "divergence":
        S, info = P.divergence(x.p, x.q, eps, x.tau, T=case["T"], grid_of_pair=goi)
    else:
        S, g, info = P.divergence_grad(x.p, x.q, eps, T=case["T"], tau=x.tau)
    out = {"cost": _scalars(x, [i["cost"] for i in info])}
    if case["tau"] != "0":
        out["S"] = _scalars(x, S)
    if op != "divergence":
        out["grad"] = g
    if op == "attribution":
        rms = P.regional_rms(g, REGIONS)
        out["rms"] = _scalars(x, np.stack([rms[k] for k in REGIONS]))
    return out


# ---------------------------------------------------------------------- work
def _applies(case):
    """Heat applies of one pass per pair or item: forward and (gradients) reverse, in halves of a transform pair."""
    T = case["T"]
    return {"smooth": 1.0, "analysis": 0.5, "synthesis": 0.5, "solve": 2.0 * T + 1, "divergence": 3 * (2.0 * T + 1),
            "gradient": 3 * (2.0 * T + 1) + 2 * (2.0 * T - 1), "attribution": 3 * (2.0 * T + 1) + 2 * (2.0 * T - 1)}[
        case["op"]]


def work(case):
    T = case["T"]
    if case["tol"]:  # the tolerance is met at the second check or so
        case = dict(case, T=min(T, 20))
    es = 8 if case["precision"] == "fp64" else 4
    ts = {"fp64": 8, "bf16": 2}.get(case["precision"], 4)
    by = fl = 0.0
    for spec, k in zip(case["grids"].split(";"), case["items"].split(";")):
        f, k = spec.split(), int(k)
        if f[0] == "hp":
            n, L = 12 * int(f[1]) ** 2, int(f[2])
            nlat, nlon = 4 * int(f[1]) - 1, 4 * int(f[1])
        else:
            nlat, nlon, L = (int(v) for v in f[1:])
            n = nlat * nlon
        h = (nlat + 1) // 2
        E = L * (L + 1) // 2 * h
        fl += k * _applies(case) * (8.0 * E + 5.0 * nlat * nlon * math.log2(nlon))
        spectrum = L * (L + 1)
        fields = {"smooth": 2 * n, "analysis": n + spectrum, "synthesis": n + spectrum, "solve": 4 * n,
                  "divergence": 2 * n, "gradient": 3 * n, "attribution": 3 * n}[case["op"]]
        by += k * fields * es
        if case["legendre"] != "recurrence":
            by += E * ts
    return {"bytes": by, "flops": fl}


# --------------------------------------------------------------------- exact
class Operator:
    """The discrete heat operator of one grid in float64: dense per-order Legendre
    matrices and FFTs (direct ring sums on HEALPix)."""

    def __init__(self, g):
        self.g = g
        L, J = g.L, g.nlat
        x = torch.as_tensor(g.x, device=DEV)
        m = torch.arange(L, device=DEV, dtype=torch.float64)[:, None]
        s = torch.sqrt(torch.clamp(1 - x * x, min=0.0))[None, :]
        Pm = torch.zeros(L, L, J, dtype=torch.float64, device=DEV)  # [m, l, j]
        diag = torch.zeros(L, J, dtype=torch.float64, device=DEV)
        diag[0] = math.sqrt(1 / (4 * math.pi))
        for k in range(1, L):
            diag[k] = diag[k - 1] * s[0] * math.sqrt((2 * k + 1) / (2 * k))
        for l in range(L):
            if l >= 1:
                a = torch.sqrt((4.0 * l * l - 1) / (l * l - m[:l] ** 2))
                r = a * x * Pm[:l, l - 1]
                if l >= 2:
                    b = torch.sqrt(((l - 1.0) ** 2 - m[:l] ** 2) / (4.0 * (l - 1) ** 2 - 1))
                    r = r - a * b * Pm[:l, l - 2]
                Pm[:l, l] = r
            Pm[l, l] = diag[l]
        self.P, self.PT = Pm, Pm.transpose(1, 2).contiguous()
        self.aw = torch.as_tensor(g.row_area, device=DEV)
        if g.kind == "hp":
            k = torch.arange(g.nlon, device=DEV, dtype=torch.float64)
            N = torch.as_tensor(g.npix.astype(np.float64), device=DEV)[:, None]
            self.valid = (k[None, :] < N).reshape(-1)
            ang = torch.as_tensor(g.phi0, device=DEV)[:, None] + 2 * math.pi * k[None, :] / N
            ph = ang[:, :, None] * torch.arange(L, device=DEV, dtype=torch.float64)
            self.W = torch.polar(torch.ones_like(ph), -ph)         # [j, k, m]
            self.WT = self.W.conj().transpose(1, 2).contiguous()   # [j, m, k]

    def analysis(self, f):
        """[B, points] -> [m, l, 2 B] (real parts of the items, then imaginary)."""
        g = self.g
        if g.kind == "hp":
            pad = torch.zeros(f.shape[0], g.nlat * g.nlon, dtype=f.dtype, device=DEV)
            pad = pad.masked_scatter(self.valid.expand_as(pad), f)
            F = torch.matmul(pad.view(-1, g.nlat, g.nlon).transpose(0, 1).to(torch.complex128), self.W)  # [j, B, m]
            F = F.permute(1, 0, 2)
        else:
            F = torch.fft.rfft(f.view(-1, g.nlat, g.nlon), dim=-1)[..., :g.L]
        F = F * self.aw[None, :, None]
        return torch.matmul(self.P, torch.cat([F.real, F.imag]).permute(2, 1, 0).contiguous())

    def synthesis(self, c):
        g = self.g
        G = torch.matmul(self.PT, c)  # [m, j, 2 B]
        B = G.shape[2] // 2
        G = torch.complex(G[..., :B], G[..., B:]).permute(2, 1, 0)  # [B, j, m]
        if g.kind == "hp":
            two = torch.full((g.L,), 2.0, dtype=torch.float64, device=DEV)
            two[0] = 1.0
            f = torch.matmul((G * two).transpose(0, 1).contiguous(), self.WT).real.transpose(0, 1)
            return f.reshape(B, -1)[:, self.valid]
        pad = torch.zeros(B, g.nlat, g.nlon // 2 + 1 - g.L, dtype=G.dtype, device=DEV)
        return (torch.fft.irfft(torch.cat([G, pad], -1), n=g.nlon, dim=-1) * g.nlon).reshape(B, -1)

    def heat(self, f, t):
        l = torch.arange(self.g.L, device=DEV, dtype=torch.float64)
        h = torch.exp(-torch.as_tensor(t, device=DEV)[None, :] * (l * (l + 1))[:, None])
        return self.synthesis(self.analysis(f) * torch.cat([h, h], 1))


def _sinkhorn(op, p, q, eps, tau, T, tol=0.0, C=10):
    """The scaling loop of [B, points] densities; returns phi, psi, cost, iterations."""
    a = op.g.area[None, :]
    t = eps / 4
    e = torch.as_tensor(eps, device=DEV)[:, None]
    bal = torch.as_tensor(np.isinf(tau), device=DEV)[:, None]
    tu = torch.as_tensor(np.where(np.isinf(tau), 1.0, tau), device=DEV)[:, None]
    lam = torch.where(bal, torch.ones_like(tu), tu / (tu + e))
    eot = e / tu
    mixed = not bool(bal.all())
    v = torch.ones_like(p)
    k = 0
    for k in range(1, T + 1):
        u = p / op.heat(v, t)
        u = u ** lam if mixed else u
        v = q / op.heat(u, t)
        v = v ** lam if mixed else v
        s = u.sum(1, keepdim=True)
        if mixed:
            c = tu / 2 * (torch.log((a * p * u ** -eot).sum(1, keepdim=True))
                          - torch.log((a * q * v ** -eot).sum(1, keepdim=True)))
            s = torch.where(bal, s, torch.exp(-c / e))
        u, v = u / s, s * v
        if tol and k % C == 0:
            if float(((u * op.heat(v, t) - p).norm(dim=1) / p.norm(dim=1)).max()) < tol:
                break
    phi, psi = e * torch.log(u), e * torch.log(v)
    cost = (a * (phi * p + psi * q)).sum(1)
    if mixed:
        un = (a * tu * ((1 - torch.exp(-phi / tu)) * p + (1 - torch.exp(-psi / tu)) * q)).sum(1)
        cost = torch.where(bal[:, 0], cost, un)
    return phi, psi, cost, k


def _divergence(op, p, q, eps, tau, T):
    """S per pair and the three costs per pair."""
    a = op.g.area[None, :]
    n = p.shape[0]
    e3, t3 = np.concatenate([eps] * 3), np.concatenate([tau] * 3)
    cost = _sinkhorn(op, torch.cat([p, p, q]), torch.cat([q, p, q]), e3, t3, T)[2].view(3, n)
    dm = (a * p).sum(1) - (a * q).sum(1)
    S = cost[0] - 0.5 * (cost[1] + cost[2]) + 0.5 * torch.as_tensor(eps, device=DEV) * dm * dm
    return S, cost


def _regional(g, grad):
    lat = np.degrees(np.arcsin(np.clip(g.x, -1, 1)))
    rows = np.repeat(np.arange(g.nlat), g.npix)
    d = grad.cpu().numpy()
    a = g.area.cpu().numpy()
    out = []
    for lo, hi in REGIONS.values():
        m = ((lat > lo + 1e-9) & (lat < hi - 1e-9))[rows]
        f = d / a
        f = f - (a * f).sum(1, keepdims=True) / a.sum()
        out.append(np.sqrt((a[m] * f[:, m] ** 2).sum(1) / a[m].sum()))
    return np.stack(out)


def exact(case, seed):
    x = Inputs(case, seed)
    op = case["op"]
    eps = 4.0 * x.t
    res, at, ct = [], 0, 0
    for gi, (g, k) in enumerate(zip(x.geoms, x.counts)):
        K = Operator(g)
        sl = slice(ct, ct + k)
        ct += k
        n = g.L * (g.L + 1) if op == "synthesis" else g.n
        p = x.p[at:at + k * n].double().view(k, n)
        q = x.q[at:at + k * n].double().view(k, n) if x.q is not None else None
        at += k * n
        il = torch.cat([torch.arange(m, g.L, device=DEV) for m in range(g.L)])
        im = torch.repeat_interleave(torch.arange(g.L, device=DEV), g.L - torch.arange(g.L, device=DEV))
        if op == "smooth":
            a = g.area[None, :]
            res.append((a * K.heat(p / a, x.t[sl]) if case["transpose"] else K.heat(p, x.t[sl])).reshape(-1))
        elif op == "analysis":
            c = K.analysis(p)[im, il]  # [(m, l), 2 k]
            res.append(torch.complex(c[:, :k], c[:, k:]).transpose(0, 1).reshape(-1))
        elif op == "synthesis":
            c = torch.zeros(g.L, g.L, 2 * k, dtype=torch.float64, device=DEV)
            pc = p.view(k, -1, 2)
            c[im, il, :k], c[im, il, k:] = pc[..., 0].transpose(0, 1), pc[..., 1].transpose(0, 1)
            res.append(K.synthesis(c).reshape(-1))
        elif op == "solve":
            res.append(_sinkhorn(K, p, q, eps[sl], x.tau[sl], case["T"], case["tol"]))
        else:
            p = p.clone().requires_grad_(op != "divergence")
            S, cost = _divergence(K, p, q, eps[sl], x.tau[sl], case["T"])
            if op != "divergence":
                S.sum().backward()
            res.append((S.detach(), cost.detach().transpose(0, 1).reshape(-1), p.grad))
        del K
    if op in ("smooth", "analysis", "synthesis"):
        return torch.cat(res)
    if op == "solve":
        return {"phi": torch.cat([r[0].reshape(-1) for r in res]), "psi": torch.cat([r[1].reshape(-1) for r in res]),
                "cost": torch.cat([r[2] for r in res]).cpu().numpy(), "iters": None}
    out = {"cost": torch.cat([r[1] for r in res]).cpu().numpy()}
    if case["tau"] != "0":
        out["S"] = torch.cat([r[0] for r in res]).cpu().numpy()
    if op != "divergence":
        out["grad"] = torch.cat([r[2].reshape(-1) for r in res])
    if op == "attribution":
        out["rms"] = _regional(x.geoms[0], res[0][2])
    return out
