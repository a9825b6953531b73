"""GPU parity of the 2D RIDC path (FP64 right-hand side + fast-diagonalisation transforms on
the matrix cores) against the FP64 oracle.

FP64: relative L2 <= 1e-12 per level.  Reduced precision (FP32 or split-BF16 transforms with
one FP64 residual refinement): a bound per level index (TOL), about 100 x the largest error
measured for that level over these cases, the full-size case and the served requests (FP32:
4.2e-15, 7.4e-16, 7.0e-16, 5.1e-16 for levels 0-3; split BF16: 1.5e-11, 2.7e-12, 3.2e-14,
3.1e-15), with the RIDC4 top level capped at 1.5e-13 = 0.1 x the discretisation error of the
1024^2 workload (1.5e-12, Richardson), the bar at which a reduced-precision result counts as
matched.  The lower levels of the split-BF16 path sit far above the top level: each level's
increment is solved to about 1e-11 of itself, and a level's error against the oracle is small
next to its own discretisation error (level 0 is first order).  Every bound holds for the
relative L2 error and for the largest pointwise error relative to the largest value.
"""
import math
import os
import sys

import numpy as np
import pytest

import workloads
from oracle import Problem, rel_l2, ridc_pipelined

pytestmark = pytest.mark.gpu

from tolerances import TOL64, tol_of  # noqa: E402  (per-level bounds, derivation above)
GOLDEN = os.path.join(os.path.dirname(__file__), "golden", "reacdiff2d_n1024_nt500.npz")


@pytest.fixture(scope="module")
def env():
    import torch
    from paper_1209_4297_amd import ridc
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    return torch, ridc


def _say(msg):
    print(msg, flush=True)
    sys.stdout.flush()


def run2d(env, prob, u0, prec="fp64", nt=None, levels=True):
    torch, ridc = env
    nt = prob["nt"] if nt is None else nt
    s = ridc.Ridc(prob, dt=prob["T"] / prob["nt"], prec=prec)
    x0 = torch.tensor(np.asarray(u0), dtype=torch.float64, device="cuda").reshape(-1)
    uT = torch.empty_like(x0)
    lv = (torch.empty(prob["order"] * x0.numel(), dtype=torch.float64, device="cuda")
          if levels else None)
    s.integrate(x0, nt, uT, lv)
    n = prob["n"]
    out = uT.cpu().numpy().reshape(n, n)
    lvs = lv.cpu().numpy().reshape(prob["order"], n, n) if levels else None
    s.close()
    return out, lvs


def errs(got, ref):
    """(relative L2, largest pointwise difference over the largest reference value)."""
    return rel_l2(got, ref), float(np.abs(got - ref).max() / np.abs(ref).max())


def oracle2d(prob, u0, nt=None):
    nt = prob["nt"] if nt is None else nt
    return ridc_pipelined(Problem.from_dict(prob), u0, nt, prob["order"])


# n = 256 and 768 (multiples of 256) run the passes that exchange prefolded planes; 768 also
# has a contraction (n/2 = 384) that is not a power of two
@pytest.mark.parametrize("n,nt,order", [(64, 40, 4), (96, 30, 4), (256, 20, 4), (160, 12, 3),
                                        (32, 8, 1), (64, 6, 6), (32, 20, 8),
                                        (192, 10, 4), (768, 6, 4)])
def test_fp64_parity(env, n, nt, order):
    prob, u0 = workloads.config_reacdiff_2d(n=n, nt=nt, order=order, T=nt * 2e-3, nu=1e-3)
    _say(f"case: 2D fp64 n={n} nt={nt} P={order}")
    ref = oracle2d(prob, u0)
    top, lvs = run2d(env, prob, u0)
    for j in range(order):
        err, emax = errs(lvs[j], ref[j])
        _say(f"  level {j}: rel L2 {err:.3e}, max {emax:.3e}")
        assert err <= TOL64 and emax <= TOL64, (j, err, emax)
    np.testing.assert_array_equal(top, lvs[-1])


@pytest.mark.parametrize("prec", ["fp32", "bf16x3"])
@pytest.mark.parametrize("n,nt", [(128, 40), (96, 20), (192, 10), (256, 12), (768, 6)])
def test_mixed_precision_parity(env, prec, n, nt):
    prob, u0 = workloads.config_reacdiff_2d(n=n, nt=nt, order=4, T=nt * 2e-3, nu=1e-3)
    _say(f"case: 2D {prec} n={n} nt={nt}")
    ref = oracle2d(prob, u0)
    top, lvs = run2d(env, prob, u0, prec=prec)
    for j in range(4):
        err, emax = errs(lvs[j], ref[j])
        _say(f"  level {j}: rel L2 {err:.3e}, max {emax:.3e}")
        assert err <= tol_of(prec, j) and emax <= tol_of(prec, j), (j, err, emax)


# the line solves: one segment row count per range of n (8 rows up to n = 512, 16 up to 1024, 32 up
# to 2048, the two-walk kernel above), at the smallest side, at the edges of the ranges and with
# segment counts that are not powers of two; nu = 1 makes r = dt nu / h^2 up to 8.7e3, so that a
# carry reaches across the whole column, nu = 0 leaves no coupling at all.  Bars: TOL64 and TOL (the
# latter was derived for nu <= 1e-3).
@pytest.mark.parametrize("n,nu,prec", [(32, 1.0, "fp64"), (96, 0.0, "fp64"), (512, 1.0, "fp64"),
                                       (544, 1e-3, "fp64"), (544, 1e-3, "bf16x3"),
                                       (1024, 1.0, "fp64"), (1056, 1.0, "fp64"),
                                       (2080, 1.0, "fp64"), (2080, 1e-3, "fp32")])
def test_line_solves_over_their_ranges(env, n, nu, prec):
    prob, u0 = workloads.config_reacdiff_2d(n=n, nt=2, order=2, T=4e-3, nu=nu)
    _say(f"case: 2D {prec} line solves n={n} nu={nu}")
    ref = oracle2d(prob, u0)
    top, lvs = run2d(env, prob, u0, prec=prec)
    for j in range(2):
        err, emax = errs(lvs[j], ref[j])
        _say(f"  level {j}: rel L2 {err:.3e}, max {emax:.3e}")
        assert err <= tol_of(prec, j) and emax <= tol_of(prec, j), (j, err, emax)


# the block tile of a pass follows the number of blocks it gives (n and the levels in a launch):
# alone and in a group a handle may take different tiles, and must keep its bits
@pytest.mark.parametrize("prec", ["fp64", "fp32", "bf16x3"])
def test_block_tiles_are_bitwise_equal(env, prec):
    torch, ridc = env
    prob, u0 = workloads.config_reacdiff_2d(n=384, nt=4, order=1, T=8e-3, nu=1e-3)
    x0 = torch.tensor(u0.reshape(-1), dtype=torch.float64, device="cuda")
    for count in (4, 15):          # 9 blocks of 128 x 128 per level: 32-, 64- and 128-tiles
        solvers = [ridc.Ridc(prob, prec=prec) for _ in range(count)]
        uTs = [torch.empty_like(x0) for _ in range(count)]
        alone = solvers[0].integrate(x0, prob["nt"]).cpu().numpy()
        ridc.integrate_batch(solvers, [x0] * count, [prob["nt"]] * count, uTs)
        torch.cuda.synchronize()
        for u in uTs:
            np.testing.assert_array_equal(u.cpu().numpy(), alone)
        for s in solvers:
            s.close()


# folded split-BF16 passes take operands folded and split by the kernels that make them: one, two and
# three slices of the contraction in the 32-tiles and, in a group, the 128-tiles (partial ones at n =
# 192 and 320), and the line solves of 32 rows a thread and of two walks.  Bars: TOL (nu <= 1e-3); a
# group's bits are those of a handle alone.
@pytest.mark.parametrize("n,count", [(64, 128), (128, 64), (192, 32), (320, 15), (1088, 1), (2112, 1)])
def test_split_operands(env, n, count):
    torch, ridc = env
    prob, u0 = workloads.config_reacdiff_2d(n=n, nt=3, order=2 if count == 1 else 1, T=6e-3, nu=1e-3)
    _say(f"case: 2D bf16x3 split operands n={n} count={count}")
    ref = oracle2d(prob, u0)
    top, lvs = run2d(env, prob, u0, prec="bf16x3")
    for j in range(prob["order"]):
        err, emax = errs(lvs[j], ref[j])
        assert err <= tol_of("bf16x3", j) and emax <= tol_of("bf16x3", j), (j, err, emax)
    if count > 1:
        x0 = torch.tensor(u0.reshape(-1), dtype=torch.float64, device="cuda")
        solvers = [ridc.Ridc(prob, prec="bf16x3") for _ in range(count)]
        uTs = [torch.empty_like(x0) for _ in range(count)]
        ridc.integrate_batch(solvers, [x0] * count, [prob["nt"]] * count, uTs)
        torch.cuda.synchronize()
        for u in uTs:
            np.testing.assert_array_equal(u.cpu().numpy().reshape(-1), np.asarray(top).reshape(-1))
        for s in solvers:
            s.close()


# small tiles with a multiple of four k-slices keep four slices' loads in flight: the smallest such sides of
# each precision and the next, alone (32-tiles), in groups of 64-tiles and in a group of 128-tiles
@pytest.mark.parametrize("n,prec", [(128, "fp64"), (256, "fp64"), (256, "fp32"), (512, "fp32"),
                                    (256, "bf16x3"), (512, "bf16x3")])
def test_four_slices_in_flight(env, n, prec):
    torch, ridc = env
    prob, u0 = workloads.config_reacdiff_2d(n=n, nt=3, order=1, T=6e-3, nu=1e-3)
    _say(f"case: 2D {prec} four slices n={n}")
    ref = oracle2d(prob, u0)
    top, lvs = run2d(env, prob, u0, prec=prec)
    err, emax = errs(lvs[0], ref[0])
    assert err <= tol_of(prec, 0) and emax <= tol_of(prec, 0), (err, emax)
    x0 = torch.tensor(u0.reshape(-1), dtype=torch.float64, device="cuda")
    tiles64, tiles128 = (n // 64) ** 2, (n // 128) ** 2
    for count in (257 // tiles64 + 1, -(-128 // tiles128)):
        solvers = [ridc.Ridc(prob, prec=prec) for _ in range(count)]
        uTs = [torch.empty_like(x0) for _ in range(count)]
        ridc.integrate_batch(solvers, [x0] * count, [prob["nt"]] * count, uTs)
        torch.cuda.synchronize()
        for u in uTs:
            np.testing.assert_array_equal(u.cpu().numpy().reshape(-1), np.asarray(top).reshape(-1))
        for s in solvers:
            s.close()


# groups of one batch run beside each other on streams of the library's own; to the caller all of it is
# in the order of its stream: inputs written just before, outputs read just after, buffers used again
@pytest.mark.parametrize("own_stream", [False, True])
def test_groups_keep_the_order_of_the_callers_stream(env, own_stream):
    torch, ridc = env
    stream = torch.cuda.Stream() if own_stream else torch.cuda.current_stream()
    shapes = [(64, "fp64"), (96, "bf16x3"), (128, "bf16x3"), (160, "fp32"), (256, "fp64"),
              (256, "bf16x3"), (64, "fp64")]
    probs = [workloads.config_reacdiff_2d(n=n, nt=5 + i, order=1 + i % 3, T=1e-2, nu=1e-3)
             for i, (n, _) in enumerate(shapes)]
    with torch.cuda.stream(stream):
        solvers = [ridc.Ridc(p, prec=prec) for (p, _), (_, prec) in zip(probs, shapes)]
        x = [torch.tensor(u.reshape(-1), dtype=torch.float64, device="cuda") for _, u in probs]
        nts = [p["nt"] for p, _ in probs]
        want = [[s.integrate(c * a, nt).clone() for s, a, nt in zip(solvers, x, nts)]
                for c in (1.0, 0.5, 0.25)]
        bufs, outs = [torch.zeros_like(a) for a in x], [torch.empty_like(a) for a in x]
        got = []
        for c in (1.0, 0.5, 0.25):
            for b, a in zip(bufs, x):
                torch.mul(a, c, out=b)
            ridc.integrate_batch(solvers, bufs, nts, outs)
            got.append([o.clone() for o in outs])
            for b in bufs:
                b.fill_(float("nan"))
    torch.cuda.synchronize()
    for w, g in zip(want, got):
        for a, b in zip(w, g):
            np.testing.assert_array_equal(b.cpu().numpy(), a.cpu().numpy())
    for s in solvers:
        s.close()


@pytest.mark.parametrize("prec", ["fp64", "bf16x3"])
def test_kernel_time_leaves_the_integration_unchanged(env, prec):
    """ridc_kernel_time runs the next step's stages again and again around its timed pass; the
    level rings and the handle's position must come out as they went in, so an integration
    timed half-way ends bitwise where an untimed one does."""
    torch, ridc = env
    prob, u0 = workloads.config_reacdiff_2d(n=256, nt=12, order=4, T=0.024, nu=1e-3)
    _say(f"case: 2D {prec} kernel_time mid-integration")
    x0 = torch.tensor(u0.reshape(-1), device="cuda")

    def run(timed):
        s = ridc.Ridc(prob, prec=prec)
        s.begin(x0, prob["nt"])
        ridc.advance([s], 8)
        if timed:
            us, flops = s.kernel_time(3)
            assert us > 0 and flops > 0
        ridc.advance([s], s.remaining())
        uT = torch.empty_like(x0)
        s.read(uT)
        s.sync()
        s.close()
        return uT.cpu().numpy()

    assert np.array_equal(run(True), run(False))


def test_largest_side_sine_mode_closed_form(env):
    """n = 16384, the largest 2D side (a vector is 2 GiB, so every address is 64-bit).  With no
    explicit term a discrete sine mode is an eigenvector of the 5-point Laplacian, and order 1
    (IMEX Euler, section II) divides it by 1 + dt nu mu each step, mu = (4/h^2)(sin^2(p pi h/2)
    + sin^2(q pi h/2)).  Sampled against that closed form.  Rounding bound: four passes of FP64
    sums of n/2 products, about 4 (n/2) eps = 3.6e-12 of the unit amplitude; checked at 1e-11.
    p != q, so a transposed axis would fail."""
    torch, ridc = env
    n, nt, p, q, nu, T = 16384, 2, 3, 5, 0.1, 0.02
    _say(f"case: 2D fp64 sine mode ({p},{q}) n={n} nt={nt} order 1")
    prob = dict(dim=2, bc="dirichlet", n=n, length=1.0, fe="none", a=0.0, nu=nu, T=T, nt=nt,
                order=1)
    h = 1.0 / (n + 1)
    idx = torch.arange(1, n + 1, dtype=torch.float64, device="cuda")
    x0 = torch.outer(torch.sin(math.pi * q * h * idx), torch.sin(math.pi * p * h * idx))
    x0 = x0.reshape(-1)                                   # row iy (mode q), column ix (mode p)
    uT = torch.empty_like(x0)
    s = ridc.Ridc(prob, dt=T / nt)
    s.integrate(x0, nt, uT)
    s.close()
    mu = 4.0 / h**2 * (math.sin(p * math.pi * h / 2) ** 2 + math.sin(q * math.pi * h / 2) ** 2)
    amp = (1.0 + (T / nt) * nu * mu) ** (-nt)
    rng = np.random.default_rng(16384)
    iy = np.concatenate([rng.integers(0, n, 2000), [0, 0, n - 1, n - 1, n // 2]])
    ix = np.concatenate([rng.integers(0, n, 2000), [0, n - 1, 0, n - 1, n // 2]])
    sel = torch.tensor(iy * n + ix, dtype=torch.int64, device="cuda")
    got = uT[sel].cpu().numpy()
    del x0, uT
    want = amp * np.sin(math.pi * q * h * (iy + 1)) * np.sin(math.pi * p * h * (ix + 1))
    err = float(np.max(np.abs(got - want)))
    _say(f"  amplitude {amp:.6f}, max abs error {err:.3e}")
    assert err <= 1e-11


def test_zero_steps_and_fixed_point(env):
    torch, ridc = env
    prob, u0 = workloads.config_reacdiff_2d(n=64, nt=10, order=4)
    top, _ = run2d(env, prob, u0, nt=0)
    np.testing.assert_array_equal(top, u0)
    # u = 0 is a fixed point of u(1-u) with zero Dirichlet data
    z = np.zeros((64, 64))
    top, lvs = run2d(env, prob, z)
    assert np.all(top == 0.0) and np.all(lvs == 0.0)


@pytest.mark.parametrize("prec", ["fp64", "fp32", "bf16x3"])
def test_batch_bitwise_equals_solo_2d(env, prec):
    torch, ridc = env
    cases = [workloads.config_reacdiff_2d(n=n, nt=nt, order=o, T=nt * 2e-3, nu=1e-3, seed=100 + n)
             for n, nt, o in [(64, 12, 4), (128, 9, 2), (64, 7, 3)]]
    solvers, u0s, uTs, solo = [], [], [], []
    for prob, u0 in cases:
        s = ridc.Ridc(prob, prec=prec)
        x0 = torch.tensor(u0.reshape(-1), dtype=torch.float64, device="cuda")
        solo.append(s.integrate(x0, prob["nt"]).cpu().numpy())
        solvers.append(s)
        u0s.append(x0)
        uTs.append(torch.empty_like(x0))
    ridc.integrate_batch(solvers, u0s, [p["nt"] for p, _ in cases], uTs)
    torch.cuda.synchronize()
    for i in range(len(cases)):
        np.testing.assert_array_equal(uTs[i].cpu().numpy(), solo[i])
    for s in solvers:
        s.close()


@pytest.mark.skipif(not os.path.exists(GOLDEN), reason="reference samples not generated")
@pytest.mark.parametrize("prec", ["fp64", "fp32", "bf16x3"])
def test_full_size_against_reference_samples(env, prec):
    """1024^2, Nt=500, order 4: the launch configuration of the full workload, checked at the
    oracle's 4096 stored sample points, norms and sums (tests/golden)."""
    ref = np.load(GOLDEN)
    prob, u0 = workloads.config_reacdiff_2d()
    _say(f"case: 2D {prec} full n=1024 nt=500")
    top, lvs = run2d(env, prob, u0, prec=prec)
    idx = ref["idx"]
    for j in range(4):
        tol = tol_of(prec, j)
        flat = lvs[j].reshape(-1)
        err, emax = errs(flat[idx], ref["samples"][j])
        nerr = abs(np.linalg.norm(flat) - ref["norms"][j]) / ref["norms"][j]
        _say(f"  level {j}: sampled rel L2 {err:.3e}, max {emax:.3e}, norm rel diff {nerr:.3e}")
        assert err <= tol and emax <= tol and nerr <= tol, (j, err, emax, nerr)
    # the result (top level): matched when within 0.1 x the RIDC4 discretisation error
    tol = tol_of(prec, 3)
    err, emax = errs(top[::8, ::8], ref["top_sub8"])
    _say(f"  top level on the 128^2 sub-grid: rel L2 {err:.3e}, max {emax:.3e}")
    assert err <= tol and emax <= tol


@pytest.mark.parametrize("prec", ["fp64", "fp32", "bf16x3"])
def test_stencil_time_bytes(env, prec):
    """The right-hand-side kernel's algorithmic bytes: every level reads its value and (j > 0)
    its j+1 window vectors, and writes the FP64 right-hand side plus a 4-byte copy in the
    reduced-precision paths."""
    torch, ridc = env
    n, P = 128, 4
    prob, u0 = workloads.config_reacdiff_2d(n=n, nt=12, order=P, T=0.02)
    s = ridc.Ridc(prob, prec=prec)
    s.begin(torch.tensor(u0.reshape(-1), dtype=torch.float64, device="cuda"), 12)
    with pytest.raises(ridc.RidcError):                    # start-up step
        s.stencil_time(3)
    ridc.advance([s], P * (P - 1) // 2)
    us, nbytes = s.stencil_time(5)
    lo = 0 if prec == "fp64" else 4
    want = sum(8 * (1 if j == 0 else j + 2) + 8 + lo for j in range(P)) * n * n
    assert us > 0 and nbytes == want
    s.sync()
    s.close()


@pytest.mark.parametrize("prec", ["fp64", "bf16x3"])
def test_graph_and_direct_launch_agree_2d(env, prec, monkeypatch):
    torch, _ = env
    prob, u0 = workloads.config_reacdiff_2d(n=128, nt=20, order=4, T=0.04, nu=1e-3)
    side = torch.cuda.Stream()
    with torch.cuda.stream(side):
        a, _ = run2d(env, prob, u0, prec, levels=False)       # captured and replayed
    direct, _ = run2d(env, prob, u0, prec, levels=False)      # null stream
    monkeypatch.setenv("RIDC_GRAPH", "0")
    with torch.cuda.stream(side):
        c, _ = run2d(env, prob, u0, prec, levels=False)
    np.testing.assert_array_equal(a, direct)
    np.testing.assert_array_equal(a, c)


def test_batch_mixing_1d_and_2d(env):
    """One batched integration over 1D and 2D instances (and two precisions) gives every
    instance the bits of its solo integration."""
    torch, ridc = env
    cases = [(workloads.config_reacdiff_2d(n=128, nt=16, order=3, T=0.03, nu=1e-3), "fp64"),
             (workloads.config_reacdiff_2d(n=96, nt=12, order=4, T=0.02, nu=1e-3), "fp32"),
             (workloads.config_reacdiff_1d(n=700, nt=30, order=4, T=0.02), "fp64"),
             (workloads.config_advdiff_1d(n=300, nt=25, order=2), "fp64")]
    solvers, u0s, uTs, solo = [], [], [], []
    for (prob, u0), prec in cases:
        s = ridc.Ridc(prob, prec=prec)
        x0 = torch.tensor(np.asarray(u0).reshape(-1), dtype=torch.float64, device="cuda")
        solo.append(s.integrate(x0, prob["nt"]).cpu().numpy())
        solvers.append(s)
        u0s.append(x0)
        uTs.append(torch.empty_like(x0))
    ridc.integrate_batch(solvers, u0s, [p["nt"] for (p, _), _ in cases], uTs)
    torch.cuda.synchronize()
    for s, uT, ref in zip(solvers, uTs, solo):
        s.sync()
        np.testing.assert_array_equal(uT.cpu().numpy(), ref)
        s.close()


# every block tile and its two forms (two slices in flight, or four where the slices are a multiple of
# four): alone 32-tiles; in a group of `c64` handles 64-tiles, of `c128` 128-tiles (order 1, so a level a
# handle).  Sides that fold with a multiple of four slices (256, 512), that fold without (192: three
# slices of split BF16, six of FP64; 384), and that do not fold (352)
@pytest.mark.parametrize("prec", ["fp64", "fp32", "bf16x3"])
@pytest.mark.parametrize("n,c64,c128", [(192, 30, 32), (256, 17, 32), (352, 9, 15), (384, 8, 15),
                                        (512, 5, 8)])
def test_64_tiles_are_bitwise_equal(env, n, c64, c128, prec):
    torch, ridc = env
    t64, t128 = ((n + 63) // 64) ** 2, ((n + 127) // 128) ** 2
    assert c64 * t64 >= 257 and c64 * t128 < 128 <= c128 * t128
    prob, u0 = workloads.config_reacdiff_2d(n=n, nt=3, order=1, T=6e-3, nu=1e-3)
    _say(f"case: 2D {prec} n={n}, {c64 * t64} blocks of 64 and {c128 * t128} of 128")
    ref = oracle2d(prob, u0)
    top, lvs = run2d(env, prob, u0, prec=prec)
    err, emax = errs(lvs[0], ref[0])
    assert err <= tol_of(prec, 0) and emax <= tol_of(prec, 0), (err, emax)
    x0 = torch.tensor(u0.reshape(-1), dtype=torch.float64, device="cuda")
    # split BF16 takes 64-tiles from 256 blocks on
    counts = [c64, c128] + ([256 // t64] if prec == "bf16x3" and 256 % t64 == 0 else [])
    for count in counts:
        solvers = [ridc.Ridc(prob, prec=prec) for _ in range(count)]
        uTs = [torch.empty_like(x0) for _ in range(count)]
        ridc.integrate_batch(solvers, [x0] * count, [prob["nt"]] * count, uTs)
        torch.cuda.synchronize()
        for u in uTs:
            np.testing.assert_array_equal(u.cpu().numpy().reshape(-1), np.asarray(top).reshape(-1))
        for s in solvers:
            s.close()


def test_batches_of_threads_that_end(env):
    """A batch of several groups forks to streams of the calling thread's.  Threads that end right after
    the call, with the work still queued, leave it whole, and their streams pass to later threads; more
    threads than idle sets are kept (8), at once and one after the other, on streams of their own."""
    import threading
    torch, ridc = env
    probs = [workloads.config_reacdiff_2d(n=n, nt=60, order=2, T=0.12, nu=1e-3) for n in (64, 96, 160)]
    want = []
    for p, u in probs:
        s = ridc.Ridc(p)
        want.append(s.integrate(torch.tensor(u.reshape(-1), device="cuda"), 60).clone())
        s.close()
    torch.cuda.synchronize()
    jobs = []

    def work():
        with torch.cuda.stream(torch.cuda.Stream()):
            solvers = [ridc.Ridc(p) for p, _ in probs]
            x = [torch.tensor(u.reshape(-1), device="cuda") for _, u in probs]
            out = [torch.empty_like(a) for a in x]
            ridc.integrate_batch(solvers, x, [60] * len(x), out)
            jobs.append((solvers, x, out))            # kept until the work has run

    for together in (12, 1, 1, 1):
        threads = [threading.Thread(target=work) for _ in range(together)]
        for t in threads:
            t.start()
        for t in threads:
            t.join()
    torch.cuda.synchronize()
    assert len(jobs) == 15
    for solvers, _, out in jobs:
        for o, w in zip(out, want):
            assert torch.equal(o, w)
        for s in solvers:
            s.close()
