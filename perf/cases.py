"""The work that programs have this library do, as cases that can be timed and checked.

A case is a dict of plain values.  ``prepare`` builds what a program holds before the call (the
initial data on the GPU and the integrator handle), ``run`` makes the one call, ``work`` counts
what it cannot do without and ``exact`` gives the same result in plain float64 torch.

Kinds of case:

``line``     one 1D integration (``Ridc.integrate``, or ``integrate_restarts`` with segments > 1)
``batch``    many ragged periodic 1D instances in one ``integrate_batch``
``plane``    one 2D integration in one of the three transform precisions
``requests`` a ``serve.Server`` that works a queue of 2D requests off
``ark``      one 1D integration with IMEX Runge-Kutta levels
``stiff``    one 1D integration whose reaction is implicit (Newton's method per stage)
"""
from __future__ import annotations

import math
import random
from fractions import Fraction

import numpy as np
import torch

TWO_PI = 2.0 * math.pi


# ---------------------------------------------------------------------------------------------
# the cases
# ---------------------------------------------------------------------------------------------
def listed():
    return [
        # the smallest call: a textbook advection-diffusion problem, all latency and launches
        dict(name="line_advect_128", kind="line", bc="periodic", n=128, length=TWO_PI,
             fe="advect", a=1.0, nu=0.1, T=1.0, nt=200, order=4, segments=1),
        # a paper-sized problem: viscous Burgers on an odd number of Dirichlet points
        dict(name="line_burgers_999", kind="line", bc="dirichlet", n=999, length=1.0,
             fe="burgers", a=0.0, nu=1e-3, T=1.0, nt=1000, order=4, segments=1),
        # a fine 1D grid over half of the usual time span
        dict(name="line_logistic_8192", kind="line", bc="dirichlet", n=8192, length=1.0,
             fe="logistic", a=0.0, nu=1e-3, T=0.5, nt=1000, order=4, segments=1),
        # a parameter study: many periodic instances of mixed sizes in one call
        dict(name="batch_256", kind="batch", count=256, nmin=256, nmax=4096, odd=False, order=4,
             T=0.05, nt=200),
        # a small 2D grid, where a step is a handful of short launches
        dict(name="plane_64_fp64", kind="plane", n=64, prec="fp64", nu=1e-3, T=0.2, nt=100,
             order=4),
        # ordinary 2D grids in the reduced-precision transforms
        dict(name="plane_256_bf16x3", kind="plane", n=256, prec="bf16x3", nu=1e-4, T=0.2, nt=100,
             order=3),
        dict(name="plane_512_fp32", kind="plane", n=512, prec="fp32", nu=1e-4, T=0.1, nt=50,
             order=2),
        # the large 2D grid, plain and with the fast transforms
        dict(name="plane_1024_fp64", kind="plane", n=1024, prec="fp64", nu=1e-4, T=0.1, nt=50,
             order=4),
        dict(name="plane_1024_bf16x3", kind="plane", n=1024, prec="bf16x3", nu=1e-4, T=0.1,
             nt=50, order=4),
        # a server that works a queue of mixed requests off
        dict(name="requests_12", kind="requests", count=12, prec="bf16x3", nmin=100, nmax=160),
        # ARK-based levels: a third-order predictor and one Euler corrector
        dict(name="ark_8192", kind="ark", bc="dirichlet", n=8192, length=1.0, fe="logistic",
             a=0.0, nu=1e-3, T=0.1, nt=200, pairs="ark3,fbe"),
        # a stiff reaction, Newton's method in every stage
        dict(name="stiff_8192", kind="stiff", n=8192, nu=1e-3, fi="cubic", kappa=1e3, T=0.05,
             nt=100, pairs="fbe,fbe,fbe,fbe"),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng: random.Random):
    kind = rng.choice(["line", "line", "batch", "plane", "plane", "plane", "requests", "ark",
                       "stiff"])
    if kind == "line":
        fe = rng.choice(["advect", "upwind", "burgers", "logistic", "none"])
        bc = "dirichlet" if fe in ("burgers", "logistic") else rng.choice(["periodic",
                                                                          "dirichlet"])
        length = TWO_PI if fe == "advect" and bc == "periodic" else 1.0
        order = rng.choice([1, 2, 3, 4, 4, 4, 5, 6, 8])
        segments = rng.choice([1, 1, 1, 2, 4])
        per = rng.randrange(max(order, 40), 160)
        return dict(kind=kind, bc=bc, n=_log(rng, 48, 8192), length=length, fe=fe,
                    a=rng.choice([-1, 1]) * round(rng.uniform(0.05, 0.2), 3),
                    nu=round(10.0 ** rng.uniform(-3.0, -2.0), 6), T=round(1e-3 * per * segments, 6),
                    nt=per * segments, order=order, segments=segments)
    if kind == "batch":
        nt = rng.randrange(40, 120)
        return dict(kind=kind, count=_log(rng, 4, 128), nmin=_log(rng, 64, 512),
                    nmax=_log(rng, 1024, 4096), odd=True, order=rng.choice([2, 3, 4, 4, 5]),
                    T=round(2.5e-4 * nt, 6), nt=nt)
    if kind == "plane":
        nt = rng.randrange(12, 50)
        return dict(kind=kind, n=32 * _log(rng, 2, 32),
                    prec=rng.choice(["fp64", "fp32", "bf16x3"]),
                    nu=round(10.0 ** rng.uniform(-5.0, -3.0), 8), T=round(2e-3 * nt, 6), nt=nt,
                    order=rng.choice([1, 2, 3, 4, 4, 6]))
    if kind == "requests":
        lo = rng.randrange(20, 80)
        return dict(kind=kind, count=rng.randrange(2, 9), prec=rng.choice(["fp32", "bf16x3"]),
                    nmin=lo, nmax=lo + rng.randrange(10, 40))
    if kind == "ark":
        fe = rng.choice(["logistic", "upwind"])
        nt = rng.randrange(30, 150)
        pairs = rng.choice(["ark3,fbe", "fbe,fbe,fbe", "ark4,ark3", "ark3", "fbe,ark3"])
        return dict(kind=kind, bc="dirichlet" if fe == "logistic" else "periodic",
                    n=_log(rng, 64, 8192), length=1.0, fe=fe, a=-0.1, nu=1e-3,
                    T=round(5e-4 * nt, 6), nt=nt, pairs=pairs)
    nt = rng.randrange(20, 80)
    fi = rng.choice(["cubic", "logistic"])
    return dict(kind=kind, n=_log(rng, 64, 8192), nu=1e-3, fi=fi,
                kappa=float(rng.randrange(50, 900 if fi == "cubic" else 200)),
                T=round(5e-4 * nt, 6), nt=nt,
                pairs=rng.choice(["fbe,fbe,fbe,fbe", "ark3,fbe", "fbe,fbe"]))


# ---------------------------------------------------------------------------------------------
# initial data (host, from the seed alone)
# ---------------------------------------------------------------------------------------------
def _grid(bc, n, length):
    if bc == "periodic":
        return np.arange(n) * (length / n)
    return np.arange(1, n + 1) * (length / (n + 1))


def _bumps(rng, n, dim):
    """Eight Gaussian bumps on [0, 1]^dim (Dirichlet points), as in a reaction front's start."""
    amp, width = rng.uniform(0.05, 1.0, 8), rng.uniform(0.01, 0.05, 8)
    x = _grid("dirichlet", n, 1.0)
    centres = rng.uniform(0.2, 0.8, (dim, 8))
    g = [np.exp(-(((x[None, :] - c[:, None]) / width[:, None]) ** 2)) for c in centres]
    return amp @ g[0] if dim == 1 else (amp[:, None] * g[1]).T @ g[0]


def _waves(rng, n, length):
    """A few long periodic waves around a mean."""
    k = np.arange(1, 9)
    alpha, beta = rng.standard_normal((2, 8)) / k**2
    phase = TWO_PI / length * np.outer(_grid("periodic", n, length), k)
    return 0.5 + np.cos(phase) @ alpha + np.sin(phase) @ beta


def _start_1d(case, rng):
    if case.get("bc", "dirichlet") == "periodic":
        return _waves(rng, case["n"], case["length"])
    if case.get("fe") == "burgers":
        x = _grid("dirichlet", case["n"], 1.0)
        a, b = rng.uniform(0.3, 1.0, 2)
        return a * np.sin(TWO_PI * x) + 0.5 * b * np.sin(math.pi * x)
    return _bumps(rng, case["n"], 1)


def _instances(case, seed):
    """The problems and initial data of a batch.  The sizes are the case's own (the same for
    every seed, so that every seed is the same amount of work); the seed draws the rest."""
    shape = random.Random(case["count"] * case["nmax"])
    rng = np.random.default_rng([seed, 4])
    out = []
    for _ in range(case["count"]):
        n = shape.choice((256, 512, 1024, 2048, 4096))
        if case["odd"]:
            n = _log(shape, case["nmin"], case["nmax"])
        prob = dict(dim=1, bc="periodic", n=n, length=TWO_PI, fe="advect",
                    a=float(rng.uniform(0.5, 2.0)), nu=float(10.0 ** rng.uniform(-3.0, -1.0)),
                    T=case["T"], nt=case["nt"], order=case["order"])
        out.append((prob, _waves(rng, n, TWO_PI)))
    return out


def _requests(case, seed):
    """The problems and initial data of a request queue.  Sides, orders and step counts are the
    case's own (the same for every seed, so that every seed is the same amount of work);
    the seed draws the diffusion coefficients and the initial data."""
    shape = random.Random(case["count"])
    rng = np.random.default_rng([seed, 5])
    out = []
    for i in range(case["count"]):
        n = (128, 256, 512, 1024)[i % 4]
        prob = dict(dim=2, bc="dirichlet", n=n, length=1.0, fe="logistic", a=0.0,
                    nu=float(10.0 ** rng.uniform(-5.0, -3.0)), T=1.0,
                    nt=shape.randrange(case["nmin"], case["nmax"] + 1),
                    order=shape.choice((2, 3, 4)))
        out.append((prob, _bumps(rng, n, 2)))
    return out


def _problem(case):
    """The workload dictionary of a single integration."""
    if case["kind"] == "plane":
        return dict(dim=2, bc="dirichlet", n=case["n"], length=1.0, fe="logistic", a=0.0,
                    nu=case["nu"], T=case["T"], nt=case["nt"], order=case["order"])
    if case["kind"] == "stiff":
        pairs = case["pairs"].split(",")
        return dict(dim=1, bc="dirichlet", n=case["n"], length=1.0, fe="none", a=0.0,
                    nu=case["nu"], T=case["T"], nt=case["nt"], order=len(pairs), pairs=pairs,
                    fi=case["fi"], kappa=case["kappa"])
    prob = dict(dim=1, bc=case["bc"], n=case["n"], length=case["length"], fe=case["fe"],
                a=case["a"], nu=case["nu"], T=case["T"], nt=case["nt"])
    if case["kind"] == "ark":
        prob["pairs"] = case["pairs"].split(",")
        prob["order"] = len(prob["pairs"])
    else:
        prob["order"] = case["order"]
    return prob


def _u0(case, seed):
    rng = np.random.default_rng([seed, 1])
    return _bumps(rng, case["n"], 2) if case["kind"] == "plane" else _start_1d(case, rng)


# ---------------------------------------------------------------------------------------------
# what a program does
# ---------------------------------------------------------------------------------------------
def _gpu(a):
    return torch.tensor(np.ascontiguousarray(a).reshape(-1), dtype=torch.float64, device="cuda")


def prepare(case, seed):
    from paper_1209_4297_amd import ridc

    state = dict(case=case)
    if case["kind"] == "batch":
        inst = _instances(case, seed)
        state["solvers"] = [ridc.Ridc(p) for p, _ in inst]
        state["nts"] = [p["nt"] for p, _ in inst]
        sizes = [p["n"] for p, _ in inst]
        state["u0s"] = list(_gpu(np.concatenate([u for _, u in inst])).split(sizes))
        state["out"] = torch.empty(sum(sizes), dtype=torch.float64, device="cuda")
        state["uTs"] = list(state["out"].split(sizes))
        return state
    if case["kind"] == "requests":
        state["requests"] = [(p, _gpu(u)) for p, u in _requests(case, seed)]
        return state
    prob = _problem(case)
    state["solver"] = ridc.Ridc(prob, prec=case.get("prec", "fp64"))
    state["u0"] = _gpu(_u0(case, seed))
    state["uT"] = torch.empty_like(state["u0"])
    return state


def run(state):
    case = state["case"]
    if case["kind"] == "batch":
        from paper_1209_4297_amd import ridc
        ridc.integrate_batch(state["solvers"], state["u0s"], state["nts"], state["uTs"])
        return state["out"]
    if case["kind"] == "requests":
        from paper_1209_4297_amd.serve import GpuExecutor, Request, Server
        server = Server(GpuExecutor(), hbm_budget=64 << 30)
        for i, (prob, u0) in enumerate(state["requests"]):
            server.submit(Request(rid=i, prob=prob, u0=u0, nsteps=prob["nt"], prec=case["prec"]))
        while not server.idle():
            server.tick()
        return [r.result for r in sorted(server.done, key=lambda r: r.rid)]
    s = state["solver"]
    if case.get("segments", 1) > 1:
        return s.integrate_restarts(state["u0"], case["nt"], case["segments"], state["uT"],
                                    sync=False)
    return s.integrate(state["u0"], case["nt"], state["uT"], sync=False)


# ---------------------------------------------------------------------------------------------
# what it cannot do without
# ---------------------------------------------------------------------------------------------
def _solve_flops(dim, n):
    """One implicit solve: two first-order sweeps in 1D, two sine transforms and sweeps in 2D."""
    return 9.0 * n if dim == 1 else n * n * (2 * 2.5 * math.log2(2 * n) + 9.0)


def _work(prob):
    """Each level's value goes through memory once a step and the level below it is read once;
    a point needs its stencil, the quadrature over the window and the solve."""
    P, n, dim = prob["order"], prob["n"], prob["dim"]
    pts = n**dim
    pairs = prob.get("pairs", ["fbe"] * P)
    implicit = dict(fbe=1, ark3=4, ark4=6)
    b = sum(8.0 * pts * (2 if j == 0 else 3) for j in range(P))
    f = sum((2 * (j + 1) + 16.0) * pts * implicit[p] + implicit[p] * _solve_flops(dim, n)
            for j, p in enumerate(pairs))
    return prob["nt"] * b, prob["nt"] * f


def work(case):
    if case["kind"] == "batch":
        probs = [p for p, _ in _instances(case, 0)]
    elif case["kind"] == "requests":
        probs = _request_shapes(case)
    else:
        probs = [_problem(case)]
    total = [_work(p) for p in probs]
    return {"bytes": sum(b for b, _ in total), "flops": sum(f for _, f in total)}


def _request_shapes(case):
    shape = random.Random(case["count"])
    out = []
    for i in range(case["count"]):
        nt = shape.randrange(case["nmin"], case["nmax"] + 1)
        out.append(dict(dim=2, n=(128, 256, 512, 1024)[i % 4], nt=nt,
                        order=shape.choice((2, 3, 4))))
    return out


# ---------------------------------------------------------------------------------------------
# the same results in plain float64 torch
# ---------------------------------------------------------------------------------------------
def _lagrange(nodes, lo, hi):
    """(values at hi, integrals over [lo, hi]) of the Lagrange basis on integer nodes."""
    val, quad = [], []
    for k in nodes:
        poly = [Fraction(1)]
        for i in nodes:
            if i != k:
                d = Fraction(1, k - i)
                poly = [(poly[e - 1] if e else 0) * d - (poly[e] if e < len(poly) else 0) * i * d
                        for e in range(len(poly) + 1)]
        val.append(float(sum(c * hi**e for e, c in enumerate(poly))))
        quad.append(float(sum(c * (hi ** (e + 1) - lo ** (e + 1)) / (e + 1)
                              for e, c in enumerate(poly))))
    return val, quad


class _Ops:
    """The grid operators of one problem; values are (..., n) or (..., n, n) tensors."""

    def __init__(self, prob, device):
        self.p, self.device = prob, device
        self.dim, self.n, self.per = prob["dim"], prob["n"], prob["bc"] == "periodic"
        n = self.n
        self.h = prob["length"] / (n if self.per else n + 1)
        self.nu_h2 = prob["nu"] / (self.h * self.h)
        self.fi, self.kappa = prob.get("fi", "diffusion"), prob.get("kappa", 0.0)
        if self.dim == 2:
            k = torch.arange(1, n + 1, dtype=torch.int64)
            s = torch.sin(math.pi * torch.arange(2 * n + 2, dtype=torch.float64) / (n + 1))
            self.Q = (math.sqrt(2.0 / (n + 1))
                      * s[torch.outer(k, k) % (2 * n + 2)]).to(device)
            mu = 4.0 * torch.sin(math.pi * k.double() / (2 * (n + 1))) ** 2
            self.mu = (mu[:, None] + mu[None, :]).to(device)
        else:
            m = n if self.per else 2 * n + 2
            k = torch.arange(m // 2 + 1, dtype=torch.float64, device=device)
            self.mu = 4.0 * torch.sin(math.pi * k / m) ** 2

    def nb(self, u, axis):
        if self.per:
            return torch.roll(u, 1, axis), torch.roll(u, -1, axis)
        z = torch.zeros_like(u.narrow(axis, 0, 1))
        n = u.shape[axis]
        return (torch.cat([z, u.narrow(axis, 0, n - 1)], axis),
                torch.cat([u.narrow(axis, 1, n - 1), z], axis))

    def lap(self, u):
        out = None
        for axis in range(-self.dim, 0):
            a, b = self.nb(u, axis)
            t = (a - u) + (b - u)
            out = t if out is None else out + t
        return self.nu_h2 * out

    def g(self, u):
        return {"diffusion": lambda: 0.0 * u, "logistic": lambda: self.kappa * (u * (1.0 - u)),
                "cubic": lambda: self.kappa * (u - u * u * u)}[self.fi]()

    def dg(self, u):
        return self.kappa * (1.0 - 2.0 * u if self.fi == "logistic" else 1.0 - 3.0 * u * u)

    def fs(self, u):
        return self.lap(u) if self.fi == "diffusion" else self.lap(u) + self.g(u)

    def fn(self, u):
        fe, a, h = self.p["fe"], self.p.get("a", 0.0), self.h
        if fe == "none":
            return torch.zeros_like(u)
        if fe == "logistic":
            return u * (1.0 - u)
        um, up = self.nb(u, -1)
        if fe == "advect":
            return -a * (up - um) / (2.0 * h)
        if fe == "upwind":
            return -a * (u - um) / h if a >= 0 else -a * (up - u) / h
        return -(up * up - um * um) / (4.0 * h)

    def solve(self, b, tau):
        """(I - tau nu Lap_h) x = b."""
        r = tau * self.nu_h2
        if self.dim == 2:
            return self.Q @ ((self.Q @ b @ self.Q) / (1.0 + r * self.mu)) @ self.Q
        if self.per:
            return torch.fft.irfft(torch.fft.rfft(b) / (1.0 + r * self.mu), n=self.n)
        z = torch.zeros_like(b[..., :1])
        e = torch.cat([z, b, z, -b.flip(-1)], -1)
        x = torch.fft.irfft(torch.fft.rfft(e) / (1.0 + r * self.mu), n=2 * self.n + 2)
        return x[..., 1:self.n + 1]

    def tridiagonal(self, diag, r, b):
        """Rows -r, diag_i, -r (zero beyond both ends), by cyclic reduction over all rows."""
        n, d, x = self.n, diag, b
        lo = torch.full_like(b, -r)
        up = lo.clone()
        lo[0] = up[-1] = 0.0
        s = 1

        def down(t, f):                              # t_{i-s}
            return torch.cat([torch.full_like(t[:s], f), t[:-s]])

        def upw(t, f):                               # t_{i+s}
            return torch.cat([t[s:], torch.full_like(t[:s], f)])

        while s < n:
            a, c = -lo / down(d, 1.0), -up / upw(d, 1.0)
            d, x, lo, up = (d + a * down(up, 0.0) + c * upw(lo, 0.0),
                            x + a * down(x, 0.0) + c * upw(x, 0.0),
                            a * down(lo, 0.0), c * upw(up, 0.0))
            s *= 2
        return x / d

    def stage(self, rhs, tau, guess):
        """y - tau f^S(y) = rhs."""
        if self.fi == "diffusion":
            y = guess
            for _ in range(2):
                y = y + self.solve(rhs - (y - tau * self.lap(y)), tau)
            return y
        y, r = guess, tau * self.nu_h2
        for _ in range(12):
            res = rhs - (y - tau * self.fs(y))
            d = self.tridiagonal(1.0 + 2.0 * r - tau * self.dg(y), r, res)
            y = y + d
            if float(d.abs().max()) < 1e-13:
                break
        return y


def _exact_ridc(prob, u0, device):
    """Level by level, every step in increment form."""
    ops, dt, nt = _Ops(prob, device), prob["T"] / prob["nt"], prob["nt"]
    prev = None
    for j in range(prob["order"]):
        u = torch.tensor(u0, dtype=torch.float64, device=device)
        traj = [u]
        if j:
            F = torch.stack([ops.fs(v) + ops.fn(v) for v in prev])
        for m in range(nt):
            if j == 0:
                u = u + ops.solve(dt * (ops.fn(u) + ops.fs(u)), dt)
            else:
                s = max(0, m + 1 - j)
                _, w = _lagrange_cached(j + 1, m - s, Fraction(1))
                q = torch.tensordot(torch.tensor(w, dtype=torch.float64, device=device),
                                    F[s:s + j + 1], 1)
                b = (u - prev[m + 1]) + dt * (q + (ops.fn(u) - ops.fn(prev[m])))
                u = prev[m + 1] + ops.solve(b, dt)
            traj.append(u)
        prev = traj
    return prev[-1]


_weights = {}


def _lagrange_cached(S, r, c):
    key = (S, r, c)
    if key not in _weights:
        _weights[key] = _lagrange(list(range(S)), Fraction(r), Fraction(r) + c)
    return _weights[key]


def _rows(text):
    return [[Fraction(x) for x in row.split()] for row in text.strip().splitlines()]


# the implicit and explicit tableaux of the pairs, and their orders
PAIRS = {
    "fbe": (_rows("0 0\n0 1"), _rows("0 0\n1 0"), 1),
    "ark3": (_rows("0 0 0 0 0\n0 1/2 0 0 0\n1/4 -5/12 2/3 0 0\n2 -7/2 1/2 2 0\n"
                   "1/6 0 2/3 -5/6 1"),
             _rows("0 0 0 0 0\n1/2 0 0 0 0\n1/4 1/4 0 0 0\n0 1 0 0 0\n1/6 0 2/3 1/6 0"), 3),
    "ark4": (_rows("0 0 0 0 0 0 0\n-1/6 1/2 0 0 0 0 0\n1/6 -1/3 1/2 0 0 0 0\n"
                   "3/8 -3/8 0 1/2 0 0 0\n1/8 0 3/8 -1/2 1/2 0 0\n-1/2 0 3 -3 1 1/2 0\n"
                   "1/6 0 0 0 2/3 -1/2 2/3"),
             _rows("0 0 0 0 0 0 0\n1/3 0 0 0 0 0 0\n1/6 1/6 0 0 0 0 0\n1/8 0 3/8 0 0 0 0\n"
                   "1/8 0 3/8 0 0 0 0\n1/2 0 -3/2 0 2 0 0\n1/6 0 0 0 2/3 1/6 0"), 4),
}


def _exact_ark(prob, u0, device):
    """Level by level: the pair of each level on the integral form of the error equation, the
    level below interpolated through S nodes."""
    ops, dt, nt = _Ops(prob, device), prob["T"] / prob["nt"], prob["nt"]
    prev, S = None, 0
    for j, name in enumerate(prob["pairs"]):
        AS, AN, order = PAIRS[name]
        S += order
        cs = [sum(row) for row in AS]
        u = torch.tensor(u0, dtype=torch.float64, device=device)
        traj = [u]
        if j:
            V = torch.stack(prev)
            F = torch.stack([ops.fs(v) + ops.fn(v) for v in prev])
        for m in range(nt):
            KS, KN, Y = [], [], u
            start = max(0, m + 2 - S)
            for i, c in enumerate(cs):
                rhs, guess, ss, sn = u, u, 0.0, 0.0
                if j:
                    li, qi = _lagrange_cached(S, m - start, c)
                    w = torch.tensor([li, qi], dtype=torch.float64, device=device)
                    e = torch.tensordot(w[0], V[start:start + S], 1)
                    rhs = rhs + dt * torch.tensordot(w[1], F[start:start + S], 1)
                    guess, ss, sn = e, ops.fs(e), ops.fn(e)
                for k in range(i):
                    rhs = rhs + dt * (float(AS[i][k]) * KS[k] + float(AN[i][k]) * KN[k])
                a = dt * float(AS[i][i])
                if a == 0.0:
                    Y = rhs
                    KS.append(ops.fs(Y) - ss)
                else:
                    rhs = rhs - a * ss
                    Y = ops.stage(rhs, a, guess)
                    KS.append((Y - rhs) / a - ss)
                KN.append(ops.fn(Y) - sn)
            u = Y
            traj.append(u)
        prev = traj
    return prev[-1]


def exact(case, seed):
    gpu = "cuda" if torch.cuda.is_available() else "cpu"
    if case["kind"] == "batch":
        # linear and periodic: the instances of one size advance together
        inst = _instances(case, seed)
        return torch.cat([_exact_modes(p, u) for p, u in inst])
    if case["kind"] == "requests":
        return [_exact_ridc(p, u, gpu).reshape(-1).cpu() for p, u in _requests(case, seed)]
    prob, u0 = _problem(case), _u0(case, seed)
    if case["kind"] == "plane":
        return _exact_ridc(prob, u0, gpu).reshape(-1).cpu()
    if case["kind"] == "line":
        for _ in range(case["segments"]):
            part = dict(prob, nt=case["nt"] // case["segments"], T=prob["T"] / case["segments"])
            u0 = _exact_ridc(part, u0, "cpu").numpy()
        return torch.tensor(u0)
    return _exact_ark(prob, u0, "cpu")


def _exact_modes(prob, u0):
    """A linear periodic instance mode by mode: its data hold no mode above 8."""
    n, dt, nt = prob["n"], prob["T"] / prob["nt"], prob["nt"]
    K = min(13, n // 2 + 1)
    k = np.arange(K)
    h = prob["length"] / n
    im = -4.0 * prob["nu"] / (h * h) * np.sin(np.pi * k / n) ** 2
    ex = -1j * prob["a"] * np.sin(TWO_PI * k / n) / h
    u = np.fft.rfft(u0)[:K]
    prev = None
    for j in range(prob["order"]):
        v, traj = u.copy(), [u]
        for m in range(nt):
            if j == 0:
                v = v + dt * (ex + im) * v / (1.0 - dt * im)
            else:
                s = max(0, m + 1 - j)
                _, w = _lagrange_cached(j + 1, m - s, Fraction(1))
                q = sum(x * y for x, y in zip(w, prev[s:s + j + 1]))
                b = (v - prev[m + 1]) + dt * ((ex + im) * q + ex * (v - prev[m]))
                v = prev[m + 1] + b / (1.0 - dt * im)
            traj.append(v)
        prev = traj
    full = np.zeros(n // 2 + 1, dtype=complex)
    full[:K] = prev[-1]
    return torch.tensor(np.fft.irfft(full, n=n))
