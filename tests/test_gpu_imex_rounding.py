"""Rounding of the IMEX level step at small r = dt nu / h^2, where every stage is solved to rounding:
the GPU's predictor against the same steps in long double, beside the FP64 oracle's own distance
from them.

The long-double steps (64-bit mantissa) take the tableau and nu / h^2 from the exact numbers and solve
every stage by FP64 solves of the long-double residual until nothing changes, so their own error is
some 1e-19.
"""
import dataclasses

import numpy as np
import pytest
import scipy.linalg

import workloads
from oracle import Problem
from oracle import ridc_ext as X
from oracle.ridc_oracle import _solve_direct

pytestmark = pytest.mark.gpu

LD = np.longdouble


@pytest.fixture(scope="module")
def env():
    import torch
    from paper_1209_4297_amd import ridc
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    return torch, ridc


def long_double_steps(p, pair, u0, nt):
    """``X.ark_integrate`` in long double (advection or no explicit term; any stiff term)."""
    tab = X.SCHEMES[pair]
    exact = lambda rows: [[LD(x.numerator) / LD(x.denominator) for x in r] for r in rows]
    AS, AN = exact(tab.AS), exact(tab.AN)
    per = p.bc == "periodic"
    h = LD(p.length) / (p.n if per else p.n + 1)
    c, dt = LD(p.nu) / (h * h), LD(p.dt)

    def shift(u, k):
        v = np.roll(u, k)
        if not per:
            v[0 if k > 0 else -1] = 0
        return v

    def fs(u):
        return c * (shift(u, 1) + shift(u, -1) - 2 * u) + X.reaction(p, u)

    def fn(u):
        return -LD(p.a) / (2 * h) * (shift(u, -1) - shift(u, 1)) if p.fe == "advect" else 0 * u

    def correction(y, res, tau):
        if p.fi == "diffusion":
            return _solve_direct(dataclasses.replace(p, dt=tau), res)
        r = tau * float(c)
        ab = np.full((3, p.n), -r)
        ab[1] = 1 + 2 * r - tau * X.reaction_prime(p, y.astype(np.float64))
        return scipy.linalg.solve_banded((1, 1), ab, res)

    y = np.asarray(u0, dtype=LD)
    for _ in range(nt):
        KS, KN = [fs(y)], [fn(y)]
        for i in range(1, tab.s):
            tau = dt * AS[i][i]
            rhs = y + dt * sum(AS[i][l] * KS[l] + AN[i][l] * KN[l] for l in range(i))
            Y = y
            for _ in range(40):
                d = correction(Y, (rhs - (Y - tau * fs(Y))).astype(np.float64), float(tau))
                Y = Y + d
                if np.abs(d).max() <= 1e-19 * np.abs(Y).max():
                    break
            KS.append((Y - rhs) / tau)
            KN.append(fn(Y))
        y = Y
    return y


def distances(env, prob, pair, u0, nt):
    """Relative L2 distance from the long-double steps of the GPU and of the oracle."""
    torch, ridc = env
    p = Problem.from_dict(prob)
    ref = long_double_steps(p, pair, u0, nt)
    s = ridc.Ridc(prob)
    gpu = s.integrate(torch.tensor(np.asarray(u0), dtype=torch.float64, device="cuda"), nt)
    s.close()
    d = [float(np.linalg.norm(v - ref) / np.linalg.norm(ref))
         for v in (gpu.cpu().numpy(), X.ark_integrate(p, pair, u0, nt))]
    print(f"case: {pair} {prob['bc']} n={prob['n']} fi={prob.get('fi')}: GPU {d[0]:.2e}, "
          f"oracle {d[1]:.2e}", flush=True)
    return d


@pytest.mark.parametrize("n", [999, 8192])
def test_newton_stage_is_as_exact_as_the_oracles(env, n):
    # one Euler stage a step, so the value's error is the solve's: the oracle solves with full FP64
    # divisions, from the same residuals and to the same stopping rule
    prob, u0 = workloads.config_stiff_1d(n=n, nt=400, order=1, fi="cubic", kappa=1e3,
                                         pairs=("fbe",))
    gpu, oracle = distances(env, prob, "fbe", u0, 60)
    assert gpu <= oracle


def test_stage_sums_round_as_often_as_the_oracles(env):
    # several stages a step: the right-hand side of a stage adds earlier stages to the value, and each
    # addition rounds it; the oracle adds the two terms of a stage at once.  r = 17, where nothing else
    # shows.  Half as much again for the different places of the other roundings
    prob, _ = workloads.config_advdiff_1d(n=8191, nt=100, order=1)
    u0 = workloads.fourier_modes_1d(8191, np.random.default_rng(8191))
    prob = dict(prob, nu=1e-3, a=0.01, T=1.0, pairs=["ark3"])
    gpu, oracle = distances(env, prob, "ark3", u0, 60)
    assert gpu <= 1.5 * oracle
