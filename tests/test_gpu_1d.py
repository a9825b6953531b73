"""GPU parity of the 1D RIDC path (fused level-step + PCR in LDS) against the FP64 oracle.

Bar: relative L2 <= 1e-12 per level against the oracle on the same seeded inputs, and the largest
pointwise difference <= 1e-12 of the largest value (both FP64; the GPU contracts to FMA and solves
by PCR, the oracle solves by FFT or banded LU, so only rounding differs).  Tiling, batching, graph replay and repetition must not change a single bit.
"""
import math
import sys

import numpy as np
import pytest

import workloads
from oracle import Problem, rel_l2, ridc_pipelined

pytestmark = pytest.mark.gpu

TOL = 1e-12


@pytest.fixture(scope="module")
def env():
    import torch
    from paper_1209_4297_amd import ridc
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    return torch, ridc


def _say(msg):
    print(msg, flush=True)
    sys.stdout.flush()


def run_gpu(env, prob, u0, nt=None, levels=True, prec="fp64", tile=None):
    torch, ridc = env
    nt = prob["nt"] if nt is None else nt
    dt = prob["T"] / prob["nt"]
    s = ridc.Ridc(prob, dt=dt, prec=prec)
    if tile is not None:
        s.set_tile(*tile)
    x0 = torch.tensor(np.asarray(u0), dtype=torch.float64, device="cuda").reshape(-1)
    uT = torch.empty_like(x0)
    lv = torch.empty(prob["order"] * x0.numel(), dtype=torch.float64, device="cuda") if levels else None
    s.integrate(x0, nt, uT, lv)
    out = uT.cpu().numpy()
    lvs = lv.cpu().numpy().reshape(prob["order"], -1) if levels else None
    s.close()
    return out, lvs


def check_against_oracle(env, prob, u0, nt=None, tol=TOL):
    nt = prob["nt"] if nt is None else nt
    _say(f"case: {prob['dim']}D {prob['bc']} n={prob['n']} P={prob['order']} nt={nt} fe={prob['fe']}")
    p = Problem(dim=prob["dim"], bc=prob["bc"], n=prob["n"], length=prob["length"], fe=prob["fe"],
                a=prob.get("a", 0.0), nu=prob["nu"], dt=prob["T"] / prob["nt"])
    ref = ridc_pipelined(p, np.asarray(u0), nt, prob["order"])
    top, lvs = run_gpu(env, prob, u0, nt)
    for j in range(prob["order"]):
        scale = np.abs(ref[j]).max()
        err = rel_l2(lvs[j], ref[j]) if scale > 0 else np.abs(lvs[j]).max()
        emax = np.abs(lvs[j] - ref[j]).max() / (scale if scale > 0 else 1.0)
        assert err <= tol and emax <= tol, (j, err, emax)
    np.testing.assert_array_equal(top, lvs[-1])
    return ref, top


def test_advdiff_n128_full(env):
    prob, u0 = workloads.config_advdiff_1d()
    ref, top = check_against_oracle(env, prob, u0)
    # and it is a fourth-order accurate answer to the semi-discrete problem (sanity)
    h = 2 * math.pi / 128
    lam = -1j * math.sin(h) / h - (4 * 0.1 / h**2) * math.sin(h / 2) ** 2
    x = np.arange(128) * h
    exact = np.imag(np.exp(lam) * np.exp(1j * x))
    assert rel_l2(top, exact) < 1e-9


def test_reacdiff_n8192_full(env):
    prob, u0 = workloads.config_reacdiff_1d()
    check_against_oracle(env, prob, u0)


def test_reacdiff_chunked_ragged(env):
    # n = 3000 with r = 4.5: few PCR stages, so the default tiling cuts it into chunks (128
    # rows, the last one ragged)
    prob, u0 = workloads.config_reacdiff_1d(n=3000, nt=400, T=0.2)
    check_against_oracle(env, prob, u0)


@pytest.mark.parametrize("order", [6, 8])
def test_long_system_default_tiling_high_orders(env, order):
    # orders 6 and 8 on a chunked system: the default tiling takes 1024 threads up to order 6
    # and 256 above, with chunks of at least 128 rows
    prob, u0 = workloads.config_reacdiff_1d(n=2304, nt=24, order=order, T=0.012)
    check_against_oracle(env, prob, u0)


@pytest.mark.parametrize("order", [1, 2, 3, 5, 6])
def test_orders(env, order):
    prob, u0 = workloads.config_advdiff_1d(n=96, nt=40, order=order, T=0.4)
    check_against_oracle(env, prob, u0)


@pytest.mark.parametrize("order", [2, 4])
def test_minimum_steps(env, order):
    prob, u0 = workloads.config_reacdiff_1d(n=64, nt=order - 1, order=order, T=0.01)
    check_against_oracle(env, prob, u0)


def test_zero_steps_returns_u0(env):
    prob, u0 = workloads.config_advdiff_1d(n=32, nt=10)
    top, lvs = run_gpu(env, prob, u0, nt=0)
    np.testing.assert_array_equal(top, u0)
    for j in range(prob["order"]):
        np.testing.assert_array_equal(lvs[j], u0)


@pytest.mark.parametrize("bc,n,fe,nu,T,nt", [
    ("periodic", 2, "advect", 0.5, 1.0, 20),      # smallest periodic cycle
    ("dirichlet", 2, "logistic", 0.1, 1.0, 20),
    ("periodic", 100, "advect", 0.05, 1.0, 50),   # non-power-of-two cycle, threshold plan
    ("periodic", 64, "none", 5.0, 1.0, 10),       # huge r: exact plan down to the 2x2 end
    ("dirichlet", 777, "advect", 1e-2, 0.5, 60),  # advection with zero ghosts
    ("dirichlet", 5000, "none", 1e-3, 1.0, 20),   # r = 1250, wrap mode on the odd extension
    ("periodic", 4096, "advect", 1e-3, 0.25, 200),
])
def test_edge_grids(env, bc, n, fe, nu, T, nt):
    length = 2 * math.pi if bc == "periodic" else 1.0
    x = workloads.grid_points(bc, n, length)
    u0 = np.sin(x) + 0.5 * np.cos(3 * x) + (0.3 if bc == "periodic" else 0.0)
    if bc == "dirichlet":
        u0 = np.clip(x * (length - x) * 3, 0, 1) + 0.1 * np.sin(7 * x)
    prob = dict(dim=1, bc=bc, n=n, length=length, fe=fe, a=0.8, nu=nu, T=T, nt=nt, order=4)
    check_against_oracle(env, prob, u0)


def test_largest_system_sine_mode_closed_form(env):
    """n = 2^28, the largest 1D system (a vector is 2 GiB; 2^21 chunks per level).  Periodic,
    no explicit term: sin(k x) is an eigenvector of the second difference, and order 1 (IMEX
    Euler, section II) divides it by 1 + 4 r sin^2(kh/2) each step, r = nu dt / h^2.  k = n/8,
    so kh = pi/4 and the mode repeats every 8 rows (built from i mod 8, exact at any i).
    Sampled against the closed form; the solve's rounding does not grow with n (a few PCR
    stages), checked at 1e-12."""
    torch, ridc = env
    n, nt, r, T = 1 << 28, 2, 0.5, 0.02
    L = 2 * math.pi
    h, dt = L / n, T / nt
    prob = dict(dim=1, bc="periodic", n=n, length=L, fe="none", a=0.0, nu=r * h * h / dt, T=T,
                nt=nt, order=1)
    _say(f"case: 1D sine mode n=2^28 nt={nt} order 1 r={r}")
    i8 = torch.arange(n, dtype=torch.int64, device="cuda") % 8
    x0 = torch.sin((math.pi / 4) * i8.to(torch.float64))
    del i8
    uT = torch.empty_like(x0)
    s = ridc.Ridc(prob, dt=dt)
    s.integrate(x0, nt, uT)
    s.close()
    amp = (1.0 + 4.0 * r * math.sin(math.pi / 8) ** 2) ** (-nt)
    rng = np.random.default_rng(1 << 28)
    idx = np.concatenate([rng.integers(0, n, 4000), [0, 1, n // 2, n - 2, n - 1]])
    got = uT[torch.tensor(idx, dtype=torch.int64, device="cuda")].cpu().numpy()
    del x0, uT
    want = amp * np.sin((math.pi / 4) * (idx % 8))
    err = float(np.max(np.abs(got - want)))
    _say(f"  amplitude {amp:.6f}, max abs error {err:.3e}")
    assert err <= 1e-12


def test_batch_bitwise_equals_solo(env):
    torch, ridc = env
    cases = workloads.config_batched_1d(count=12, nt=120, T=0.03)
    solvers, u0s, uTs, solo = [], [], [], []
    for prob, u0 in cases:
        s = ridc.Ridc(prob)
        x0 = torch.tensor(u0, dtype=torch.float64, device="cuda")
        solo.append(s.integrate(x0, prob["nt"]).cpu().numpy())
        solvers.append(s)
        u0s.append(x0)
        uTs.append(torch.empty_like(x0))
    # mix in a Dirichlet reaction-diffusion instance of another order
    prob2, u02 = workloads.config_reacdiff_1d(n=2500, nt=90, order=3, T=0.05)
    s2 = ridc.Ridc(prob2)
    x2 = torch.tensor(u02, dtype=torch.float64, device="cuda")
    solo.append(s2.integrate(x2, prob2["nt"]).cpu().numpy())
    solvers.append(s2)
    u0s.append(x2)
    uTs.append(torch.empty_like(x2))
    nts = [p["nt"] for p, _ in cases] + [prob2["nt"]]
    ridc.integrate_batch(solvers, u0s, nts, uTs)
    torch.cuda.synchronize()
    for i, uT in enumerate(uTs):
        np.testing.assert_array_equal(uT.cpu().numpy(), solo[i])
    # stepping interface with uneven chunks gives the same bits too
    for s, x0, prob_nt in zip(solvers, u0s, nts):
        s.begin(x0, prob_nt)
    while any(s.remaining() > 0 for s in solvers):
        ridc.advance(solvers, 37)
    for i, s in enumerate(solvers):
        out = torch.empty_like(u0s[i])
        s.read(out)
        s.sync()
        np.testing.assert_array_equal(out.cpu().numpy(), solo[i])
    for s in solvers:
        s.close()


@pytest.mark.parametrize("policy", [(256, 0), (512, 512), (1024, 768), (256, 1024), (1024, 0),
                                    "tuned"])
def test_batch_tilings_are_bitwise_identical(env, policy):
    """Grouped launches cut long cycles into chunks, change the thread count, and use the
    kernels specialised for the batch's highest order; none of it may change a bit."""
    torch, ridc = env
    cases = workloads.config_batched_1d(count=10, nt=60, T=0.015)
    prob2, u02 = workloads.config_reacdiff_1d(n=2500, nt=50, order=3, T=0.03)
    prob3, _ = workloads.config_advdiff_1d(n=512, nt=40, order=7, T=0.05)   # levels up to 6
    u03 = workloads.fourier_modes_1d(512, np.random.default_rng(7))
    cases = cases + [(prob2, u02), (prob3, u03)]
    solvers, u0s, uTs, solo = [], [], [], []
    for prob, u0 in cases:
        s = ridc.Ridc(prob)
        x0 = torch.tensor(u0, dtype=torch.float64, device="cuda")
        solo.append(s.integrate(x0, prob["nt"]).cpu().numpy())
        solvers.append(s)
        u0s.append(x0)
        uTs.append(torch.empty_like(x0))
    nts = [p["nt"] for p, _ in cases]
    try:
        if policy == "tuned":
            t, r = ridc.autotune_batch(solvers)
            _say(f"batch tiling chosen: threads {t}, rows {r}")
        else:
            ridc.set_batch_tile(*policy)
        ridc.integrate_batch(solvers, u0s, nts, uTs)
        torch.cuda.synchronize()
        for i, uT in enumerate(uTs):
            np.testing.assert_array_equal(uT.cpu().numpy(), solo[i])
    finally:
        ridc.set_batch_tile(256, 0)
        for s in solvers:
            s.close()


def test_graph_and_direct_launch_agree(env, monkeypatch):
    """On a stream of its own an integration is captured in a HIP graph and replayed (a second
    call replays the cached graph); it must give the bits of direct launches, on that stream
    with capture switched off and on the null stream."""
    torch, _ = env
    prob, u0 = workloads.config_reacdiff_1d(n=2048, nt=300, T=0.15)
    side = torch.cuda.Stream()
    with torch.cuda.stream(side):
        a, _ = run_gpu(env, prob, u0, levels=False)          # captured
        b, _ = run_gpu(env, prob, u0, levels=False)
    direct, _ = run_gpu(env, prob, u0, levels=False)          # null stream: direct launches
    monkeypatch.setenv("RIDC_GRAPH", "0")
    with torch.cuda.stream(side):
        c, _ = run_gpu(env, prob, u0, levels=False)
    np.testing.assert_array_equal(a, b)
    np.testing.assert_array_equal(a, c)
    np.testing.assert_array_equal(a, direct)


def test_graph_replay_of_one_handle(env):
    """One handle integrating twice on its own stream replays its cached graph."""
    torch, ridc = env
    prob, u0 = workloads.config_advdiff_1d(n=256, nt=60)
    side = torch.cuda.Stream()
    with torch.cuda.stream(side):
        s = ridc.Ridc(prob)
        x0 = torch.tensor(u0, dtype=torch.float64, device="cuda")
        first = s.integrate(x0, 60).clone()
        second = s.integrate(x0, 60)
        side.synchronize()
        s.close()
    alone, _ = run_gpu(env, prob, u0, levels=False)
    np.testing.assert_array_equal(first.cpu().numpy(), alone)
    np.testing.assert_array_equal(second.cpu().numpy(), alone)


def test_nonfinite_is_reported(env):
    torch, ridc = env
    prob, u0 = workloads.config_advdiff_1d(n=64, nt=20)
    u0 = u0.copy()
    u0[5] = np.nan
    s = ridc.Ridc(prob)
    x0 = torch.tensor(u0, dtype=torch.float64, device="cuda")
    with pytest.raises(ridc.RidcError) as ei:
        s.integrate(x0, 20)
    assert ei.value.code == ridc.RIDC_E_NONFINITE
    # the handle stays usable
    out = s.integrate(torch.tensor(workloads.config_advdiff_1d(n=64, nt=20)[1], dtype=torch.float64,
                                   device="cuda"), 20)
    assert torch.isfinite(out).all()
    s.close()


def test_batch_reports_nonfinite_per_instance(env):
    """A batched integration flags the instance whose result is not finite, and only it."""
    torch, ridc = env
    cases = [workloads.config_advdiff_1d(n=n, nt=20) for n in (64, 256, 100)]
    solvers = [ridc.Ridc(p) for p, _ in cases]
    u0s = [torch.tensor(u, dtype=torch.float64, device="cuda") for _, u in cases]
    u0s[1][17] = float("nan")
    uTs = [torch.empty_like(x) for x in u0s]
    ridc.integrate_batch(solvers, u0s, [20, 20, 20], uTs)
    solvers[0].sync()
    solvers[2].sync()
    with pytest.raises(ridc.RidcError) as ei:
        solvers[1].sync()
    assert ei.value.code == ridc.RIDC_E_NONFINITE
    for i in (0, 2):
        alone = solvers[i].integrate(u0s[i], 20)
        assert torch.equal(alone, uTs[i])
    for s in solvers:
        s.close()


def test_state_errors(env):
    torch, ridc = env
    prob, u0 = workloads.config_advdiff_1d(n=64, nt=20)
    s = ridc.Ridc(prob)
    x0 = torch.tensor(u0, dtype=torch.float64, device="cuda")
    out = torch.empty_like(x0)
    with pytest.raises(ridc.RidcError) as ei:
        s.read(out)
    assert ei.value.code == ridc.RIDC_E_STATE
    s.begin(x0, 20)
    assert s.remaining() == 20 + 6
    with pytest.raises(ridc.RidcError):
        s.read(out)
    with pytest.raises(ridc.RidcError) as ei:
        s.begin(x0, 2)                      # below order - 1
    assert ei.value.code == ridc.RIDC_E_INVAL
    s.close()


def test_tilings_are_bitwise_identical(env):
    torch, ridc = env
    prob, u0 = workloads.config_reacdiff_1d(n=2048, nt=120, T=0.06)
    x0 = torch.tensor(u0, dtype=torch.float64, device="cuda")
    s = ridc.Ridc(prob)
    outs = []
    tiles = [(256, 0, 0), (1024, 0, 1), (256, 1024, 0), (512, 512, 1), (128, 2048, 0),
             (1024, 256, 1), (512, 0, 2), (1024, 0, 2)]
    for threads, rows, flags in tiles:
        try:
            s.set_tile(threads, rows, flags)
        except ridc.RidcError:
            continue
        _say(f"tile threads={threads} rows={rows} flags={flags}")
        outs.append(s.integrate(x0, prob["nt"]).cpu().numpy())
    assert len(outs) >= 6
    for o in outs[1:]:
        np.testing.assert_array_equal(o, outs[0])
    t, r, f = s.autotune()
    _say(f"autotuned: threads={t} rows={r} flags={f}")
    np.testing.assert_array_equal(s.integrate(x0, prob["nt"]).cpu().numpy(), outs[0])
    s.close()


@pytest.mark.parametrize("bc,n,order,nt", [("periodic", 1000, 4, 50), ("dirichlet", 999, 4, 40),
                                           ("periodic", 2048, 4, 30), ("dirichlet", 3000, 3, 30),
                                           ("periodic", 128, 1, 20), ("dirichlet", 64, 6, 25),
                                           ("periodic", 4096, 2, 40), ("periodic", 128, 4, 60),
                                           ("dirichlet", 200, 4, 30)])
def test_fused_integration_equals_per_step_kernel(env, bc, n, order, nt):
    """Systems that fit one CU run their whole integration in one workgroup; the result is
    bitwise that of one launch per pipeline step."""
    torch, ridc = env
    length = 2 * math.pi if bc == "periodic" else 1.0
    x = workloads.grid_points(bc, n, length)
    u0 = np.sin(x) + 0.25 * np.cos(5 * x) if bc == "periodic" else x * (length - x) * 4
    prob = dict(dim=1, bc=bc, n=n, length=length, fe="advect" if bc == "periodic" else "logistic",
                a=0.6, nu=2e-3, T=0.05, nt=nt, order=order)
    _say(f"case: fused vs per-step {bc} n={n} P={order} nt={nt}")
    step, lv_s = run_gpu(env, prob, u0)
    fused, lv_f = run_gpu(env, prob, u0, tile=(512, 0, 2))
    if order <= 4:
        fused2, _ = run_gpu(env, prob, u0, tile=(1024, 0, 2))
        np.testing.assert_array_equal(fused2, step)
    else:                                   # the 1024-thread workgroup covers orders <= 4
        with pytest.raises(ridc.RidcError) as ei:
            run_gpu(env, prob, u0, tile=(1024, 0, 2))
        assert ei.value.code == ridc.RIDC_E_INVAL
    np.testing.assert_array_equal(fused, step)
    np.testing.assert_array_equal(lv_f, lv_s)
    p = Problem(dim=1, bc=bc, n=n, length=length, fe=prob["fe"], a=0.6, nu=2e-3, dt=0.05 / nt)
    ref = ridc_pipelined(p, u0, nt, order)[-1]
    assert rel_l2(fused, ref) <= TOL


def test_batch_kernel_time_and_its_errors(env):
    torch, ridc = env
    cases = workloads.config_batched_1d(count=6, nt=40, T=0.01)
    solvers = [ridc.Ridc(p) for p, _ in cases]
    x0s = [torch.tensor(u, dtype=torch.float64, device="cuda") for _, u in cases]
    try:
        with pytest.raises(ridc.RidcError) as ei:          # not armed
            ridc.batch_kernel_time(solvers, 5)
        assert ei.value.code == ridc.RIDC_E_STATE
        for s, x0, (p, _) in zip(solvers, x0s, cases):
            s.begin(x0, p["nt"])
        with pytest.raises(ridc.RidcError) as ei:          # start-up step: not every level active
            ridc.batch_kernel_time(solvers, 5)
        assert ei.value.code == ridc.RIDC_E_STATE
        ridc.advance(solvers, 6)
        us, nbytes = ridc.batch_kernel_time(solvers, 10)
        assert us > 0
        assert nbytes == sum(s.step_cost()[0] for s in solvers)
        # the handles did not advance: the integration finishes with the solo bits
        while any(s.remaining() > 0 for s in solvers):
            ridc.advance(solvers, 64)
        for s, x0, (p, _) in zip(solvers, x0s, cases):
            out = torch.empty_like(x0)
            s.read(out)
            s.sync()
            solo = ridc.Ridc(p)
            np.testing.assert_array_equal(out.cpu().numpy(), solo.integrate(x0, p["nt"]).cpu().numpy())
            solo.close()
    finally:
        for s in solvers:
            s.close()


def test_stencil_time_is_2d_only(env):
    torch, ridc = env
    prob, u0 = workloads.config_advdiff_1d(n=64, nt=20)
    s = ridc.Ridc(prob)
    s.begin(torch.tensor(u0, dtype=torch.float64, device="cuda"), 20)
    with pytest.raises(ridc.RidcError) as ei:
        s.stencil_time(5)
    assert ei.value.code == ridc.RIDC_E_UNSUPPORTED
    s.close()


@pytest.mark.parametrize("order", [1, 2, 4, 5, 6])
@pytest.mark.parametrize("bc,fe", [("periodic", "advect"), ("periodic", "upwind"),
                                   ("dirichlet", "burgers"), ("dirichlet", "logistic"),
                                   ("dirichlet", "none")])
def test_small_systems_in_one_workgroup(env, order, bc, fe):
    """Up to 256 rows a handle of its own, or a batch of such handles, runs whole ranges of steps in
    one workgroup with a wave a level.  Sizes around one, two and four rows a lane; the bits are those
    of a launch per step whatever the range is cut into, alone and in a batch, and the oracle agrees."""
    torch, ridc = env
    nt = 18
    solvers, u0s, nts, want = [], [], [], []
    for n in (2, 3, 7, 63, 64, 65, 127, 128, 129, 192, 255, 256):
        _say(f"case: small {bc} {fe} n={n} P={order}")
        length = 2 * math.pi if bc == "periodic" else 1.0
        x = workloads.grid_points(bc, n, length)
        u0 = np.sin(x) + 0.25 * np.cos(5 * x) if bc == "periodic" else x * (length - x) * 4
        prob = dict(dim=1, bc=bc, n=n, length=length, fe=fe, a=0.6, nu=2e-3, T=0.05, nt=nt,
                    order=order)
        small, lv = run_gpu(env, prob, u0)
        step, lv_s = run_gpu(env, prob, u0, tile=(256, 0, 0))
        np.testing.assert_array_equal(small, step)
        np.testing.assert_array_equal(lv, lv_s)
        p = Problem(dim=1, bc=bc, n=n, length=length, fe=fe, a=0.6, nu=2e-3, dt=0.05 / nt)
        ref = ridc_pipelined(p, u0, nt, order)
        for j in range(order):
            assert rel_l2(lv[j], ref[j]) <= TOL
        s = ridc.Ridc(prob)
        x0 = torch.tensor(u0, dtype=torch.float64, device="cuda")
        out = torch.empty_like(x0)
        s.begin(x0, nt)
        chunk = 1
        while s.remaining() > 0:
            ridc.advance([s], chunk)
            chunk = chunk % 5 + 2
            if chunk == 4:                       # the rings pass to the other kernel and back
                s.set_tile(256, 0, 0)
            elif chunk == 5 and order <= 6:
                s.set_tile(512, 0, 2)
        s.read(out)
        s.sync()
        np.testing.assert_array_equal(out.cpu().numpy(), step)
        s.close()
        s = ridc.Ridc(prob)
        solvers.append(s)
        u0s.append(x0)
        nts.append(nt - (n % 3))
        want.append(run_gpu(env, dict(prob), u0, nt=nts[-1], tile=(256, 0, 0))[0])
    uTs = [torch.empty_like(x0) for x0 in u0s]
    ridc.integrate_batch(solvers, u0s, nts, uTs)
    torch.cuda.synchronize()
    for uT, w in zip(uTs, want):
        np.testing.assert_array_equal(uT.cpu().numpy(), w)
    for s in solvers:
        s.close()


@pytest.mark.parametrize("bc,n,order", [("periodic", 257, 4), ("dirichlet", 300, 1),
                                        ("dirichlet", 129, 8), ("periodic", 200, 7),
                                        ("periodic", 999, 6), ("dirichlet", 2047, 4),
                                        ("periodic", 1500, 8), ("periodic", 9500, 2)])
@pytest.mark.parametrize("nu", [2e-5, 2e-3, 2e-1])
def test_default_tilings_equal_whole_cycles(env, bc, n, order, nu):
    """Chunks (their number depends on the halo, so on nu) or a whole cycle, as a new handle takes
    them, give the bits of one 256-thread workgroup a level."""
    length = 2 * math.pi if bc == "periodic" else 1.0
    x = workloads.grid_points(bc, n, length)
    u0 = np.sin(x) + 0.25 * np.cos(5 * x) if bc == "periodic" else x * (length - x) * 4
    nt = 12
    prob = dict(dim=1, bc=bc, n=n, length=length, fe="advect" if bc == "periodic" else "logistic",
                a=0.6, nu=nu, T=0.004, nt=nt, order=order)
    _say(f"case: default tile {bc} n={n} P={order} nu={nu}")
    got, lv = run_gpu(env, prob, u0)
    want, lv_w = run_gpu(env, prob, u0, tile=(256, 0, 0))
    np.testing.assert_array_equal(got, want)
    np.testing.assert_array_equal(lv, lv_w)


def _step_time(env, s, x0, k):
    """Least time of a pipeline step, us, over runs of advances by k steps."""
    import time
    torch, ridc = env
    s.begin(x0, 10**6)
    ridc.advance([s], 100)
    best = 1e30
    for _ in range(10):
        torch.cuda.synchronize()
        t = time.perf_counter()
        for _ in range(240 // k):
            ridc.advance([s], k)
        torch.cuda.synchronize()
        best = min(best, (time.perf_counter() - t) / (240 // k * k))
    return best * 1e6


@pytest.mark.parametrize("n,order", [(64, 4), (128, 6), (256, 1), (256, 4), (256, 6)])
def test_short_ranges_of_small_systems(env, n, order):
    """A handle advanced a step or a few at a time (serving) costs no more than launches per step: the
    whole-range workgroup, which loads and stores all rings, takes the ranges that pay for it (it cost up
    to 3.3 times a step).  A third above is left for the spread of the timing."""
    torch, ridc = env
    ridc.tune_clear()                    # nothing recorded by other tests
    x = workloads.grid_points("periodic", n, 2 * math.pi)
    x0 = torch.tensor(np.sin(x), dtype=torch.float64, device="cuda")
    prob = dict(dim=1, bc="periodic", n=n, length=2 * math.pi, fe="advect", a=0.6, nu=2e-3, T=0.05,
                nt=1000, order=order)
    s, per_step = ridc.Ridc(prob), ridc.Ridc(prob)
    per_step.set_tile(256, 0, 0)
    for k in (1, 2, 3):
        a, b = _step_time(env, s, x0, k), _step_time(env, per_step, x0, k)
        _say(f"case: n={n} P={order} ranges of {k}: {a:.2f} us a step, per-step launches {b:.2f}")
        assert a <= 1.33 * b
    s.close()
    per_step.close()


def test_a_batch_takes_all_the_steps_there_are(env):
    """The largest max_steps advances every instance to its end, also after a first advance."""
    torch, ridc = env
    for sizes in ((64, 100), (100, 300)):          # whole ranges in one workgroup; grouped launches
        solvers, x0s, want = [], [], []
        for n in sizes:
            x = workloads.grid_points("periodic", n, 2 * math.pi)
            x0s.append(torch.tensor(np.sin(x), dtype=torch.float64, device="cuda"))
            prob = dict(dim=1, bc="periodic", n=n, length=2 * math.pi, fe="advect", a=0.6, nu=2e-3,
                        T=0.05, nt=20, order=3)
            solvers.append(ridc.Ridc(prob))
            want.append(solvers[-1].integrate(x0s[-1], 20).clone())
        for s, x0 in zip(solvers, x0s):
            s.begin(x0, 20)
        ridc.advance(solvers, 3)
        ridc.advance(solvers, 2**63 - 1)
        for s, x0, w in zip(solvers, x0s, want):
            assert s.remaining() == 0
            out = torch.empty_like(x0)
            s.read(out)
            s.sync()
            assert torch.equal(out, w)
            s.close()


def test_long_ranges_of_a_batch_go_by_several_launches(env):
    """Instances with more steps than one launch of small systems takes (65536), less and just as many,
    in a batch: the same bits as launches per step."""
    torch, ridc = env
    solvers, x0s, nts, want = [], [], [], []
    for n, nt in ((5, 65536 + 700), (2, 65536 - 1), (7, 65536), (3, 900), (5, 2 * 65536 + 1)):
        x = workloads.grid_points("periodic", n, 2 * math.pi)
        prob = dict(dim=1, bc="periodic", n=n, length=2 * math.pi, fe="advect", a=0.6, nu=2e-3,
                    T=1e-4 * nt, nt=nt, order=2)
        u0 = 0.5 + np.cos(x)
        want.append(run_gpu(env, prob, u0, tile=(256, 0, 0))[0])
        solvers.append(ridc.Ridc(prob))
        x0s.append(torch.tensor(u0, dtype=torch.float64, device="cuda"))
        nts.append(nt)
    uTs = [torch.empty_like(x0) for x0 in x0s]
    ridc.integrate_batch(solvers, x0s, nts, uTs)
    torch.cuda.synchronize()
    for s, uT, w in zip(solvers, uTs, want):
        np.testing.assert_array_equal(uT.cpu().numpy(), w)
        s.close()


@pytest.mark.parametrize("count", [1, 3])
def test_kernel_time_of_small_systems(env, count):
    """The timing of an untuned small system (or a batch of them) is that of the kernel its ranges run,
    a third of a launch per step; it takes more steps than are left and leaves the handles armed and the
    integration's bits alone."""
    torch, ridc = env
    ridc.tune_clear()                    # nothing recorded by other tests
    x = workloads.grid_points("periodic", 128, 2 * math.pi)
    x0 = torch.tensor(np.sin(x), dtype=torch.float64, device="cuda")
    prob = dict(dim=1, bc="periodic", n=128, length=2 * math.pi, fe="advect", a=0.6, nu=2e-3, T=0.05,
                nt=30, order=4)
    solvers = [ridc.Ridc(prob) for _ in range(count)]
    want = solvers[0].integrate(x0, 30).cpu().numpy()
    for s in solvers:
        s.begin(x0, 30)
    ridc.advance(solvers, 10)
    us, nbytes = ridc.batch_kernel_time(solvers, 200) if count > 1 else solvers[0].kernel_time(200)
    assert nbytes == sum(s.step_cost()[0] for s in solvers)
    per_step = ridc.Ridc(prob)
    per_step.set_tile(256, 0, 0)
    per_step.begin(x0, 30)
    ridc.advance([per_step], 10)
    launch = per_step.kernel_time(200)[0]
    _say(f"case: {count} small systems {us:.2f} us a step, launches per step {launch:.2f}")
    assert us < 0.7 * launch
    while any(s.remaining() > 0 for s in solvers):
        ridc.advance(solvers, 7)
    for s in solvers:
        out = torch.empty_like(x0)
        s.read(out)
        s.sync()
        np.testing.assert_array_equal(out.cpu().numpy(), want)
        s.close()
    per_step.close()


def _small_step(env, order):
    """(us a step of an untouched handle's timing, launches per step) at n = 200."""
    torch, ridc = env
    x = workloads.grid_points("periodic", 200, 2 * math.pi)
    x0 = torch.tensor(np.sin(x), dtype=torch.float64, device="cuda")
    prob = dict(dim=1, bc="periodic", n=200, length=2 * math.pi, fe="advect", a=0.6, nu=2e-3, T=0.05,
                nt=400, order=order)
    out = []
    for tile in (None, (256, 0, 0)):
        s = ridc.Ridc(prob)
        if tile:
            s.set_tile(*tile)
        s.begin(x0, 400)
        ridc.advance([s], 20)
        out.append(s.kernel_time(100)[0])
        s.close()
    return out


def test_other_orders_records_leave_small_systems_alone(env, tmp_path):
    """A tiling measured at one order is not another order's: after an order 8 handle's, and with a file's
    entry for all orders that does not fit this one, a small system still runs whole ranges."""
    import json
    torch, ridc = env
    ridc.tune_clear()
    prob = dict(dim=1, bc="periodic", n=200, length=2 * math.pi, fe="advect", a=0.6, nu=2e-3, T=0.05,
                nt=400, order=8)
    s = ridc.Ridc(prob)
    s.autotune()
    s.close()
    small, launch = _small_step(env, 4)
    _say(f"case: order 4 after order 8's record: {small:.2f} us, launches per step {launch:.2f}")
    assert small < 0.8 * launch
    path = tmp_path / "tune.json"
    ridc.tune_save(str(path))
    doc = json.loads(path.read_text())
    (rec,) = doc["tile1d"]
    assert rec["n"] == 200 and rec["order"] == 8
    del rec["order"]                              # as an older file has it
    rec.update(threads=1024, rows=0, flags=2)     # a whole range in 1024 threads: orders up to 4
    path.write_text(json.dumps(doc))
    ridc.tune_clear()
    ridc.tune_load(str(path))
    small, launch = _small_step(env, 6)
    _say(f"case: order 6 beside order 4's whole range: {small:.2f} us, launches per step {launch:.2f}")
    assert small < 0.8 * launch
    ridc.tune_clear()


@pytest.mark.parametrize("n", [65536, 65537, 200000])
def test_long_systems_of_high_order(env, n):
    """The default tiling of a long system of order 8 takes no longer than either thread count it chooses
    from (it took 1.28 times as long at n = 200000), and the bits are theirs."""
    import time
    torch, ridc = env
    ridc.tune_clear()
    x = workloads.grid_points("periodic", n, 2 * math.pi)
    x0 = torch.tensor(np.sin(x), dtype=torch.float64, device="cuda")
    h = 2 * math.pi / n
    prob = dict(dim=1, bc="periodic", n=n, length=2 * math.pi, fe="advect", a=0.01, nu=3.0 * h * h / 1e-4,
                T=6e-3, nt=60, order=8)
    times, outs = [], []
    stream = torch.cuda.Stream()
    with torch.cuda.stream(stream):
        for tile in (None, (256, 1024, 0), (512, 1024, 0)):
            s = ridc.Ridc(prob)
            if tile:
                s.set_tile(*tile)
            outs.append(s.integrate(x0, 60).clone())
            best = 1e30
            for _ in range(8):
                t = time.perf_counter()
                s.integrate(x0, 60, outs[-1])
                best = min(best, time.perf_counter() - t)
            times.append(best * 1e6 / 88)
            s.close()
    _say(f"case: order 8 n={n}: default {times[0]:.1f} us a step, 256 threads {times[1]:.1f}, 512 "
         f"{times[2]:.1f}")
    assert torch.equal(outs[0], outs[1]) and torch.equal(outs[0], outs[2])
    assert times[0] <= 1.1 * min(times[1:])


def _periodic_batch(ridc, torch, sizes, halo, order=4, nt=40):
    """Handles and initial data of periodic systems whose PCR halo is `halo` rows or the longest that
    their side has below it."""
    solvers, x0s = [], []
    dt = 1e-4
    for n in sizes:
        r = max(10.0 ** e for e in np.linspace(-2, 8, 200)
                if 2 ** ridc.pcr_plan(10.0 ** e, n)[0] - 1 <= halo)
        h = 2 * math.pi / n
        prob = dict(dim=1, bc="periodic", n=n, length=2 * math.pi, fe="advect", a=0.01,
                    nu=r * h * h / dt, T=dt * nt, nt=nt, order=order)
        x = workloads.grid_points("periodic", n, 2 * math.pi)
        solvers.append(ridc.Ridc(prob))
        x0s.append(torch.tensor(np.sin(x) + 0.3 * np.cos(3 * x), dtype=torch.float64, device="cuda"))
    return solvers, x0s


def test_default_grouped_tiling_with_long_halos(env):
    """128 instances of 700 to 1400 rows with halos of 255: the automatic tiling takes no longer than whole
    cycles (chunks that recompute two rows of three took 1.6 times as long)."""
    import time
    torch, ridc = env
    sizes = [int(v) for v in np.random.default_rng(0).integers(700, 1400, 128)]
    nt = 40
    solvers, x0s = _periodic_batch(ridc, torch, sizes, 255, nt=nt)
    uTs = [torch.empty_like(a) for a in x0s]
    times = []
    try:
        for tile in (None, (512, 0)):
            ridc.tune_clear()
            if tile:
                ridc.set_batch_tile(*tile)
            best = 1e30
            for _ in range(6):
                torch.cuda.synchronize()
                t = time.perf_counter()
                ridc.integrate_batch(solvers, x0s, [nt] * len(sizes), uTs)
                torch.cuda.synchronize()
                best = min(best, time.perf_counter() - t)
            times.append(best * 1e6 / (nt + 6))
    finally:
        ridc.tune_clear()
        for s in solvers:
            s.close()
    _say(f"case: 128 instances, halo 255: automatic {times[0]:.1f} us a step, whole cycles {times[1]:.1f}")
    assert times[0] <= 1.1 * times[1]


# the automatic tiling of a grouped launch goes by the rows it covers: from 8e5 (256, 1536), from 2e5 (512,
# 768), from 5e4 (512, 512), below (512, 384); instances of odd sides, at the lower edge of each and at the
# least there is, with halos that give chunks and halos that leave whole cycles
@pytest.mark.parametrize("halo", [31, 127, 255, 511])
@pytest.mark.parametrize("count,lo,hi", [(61, 3000, 4000), (40, 1100, 1700), (13, 900, 1200),
                                         (9, 300, 700), (2, 257, 300)])
def test_automatic_grouped_tilings_are_bitwise_solo(env, count, lo, hi, halo):
    torch, ridc = env
    rng = np.random.default_rng(count)
    sizes = [int(v) for v in rng.integers(lo, hi, count)]
    _say(f"case: {count} instances, {4 * sum(sizes)} rows of all levels, halo {halo}")
    ridc.tune_clear()
    solvers, x0s = _periodic_batch(ridc, torch, sizes, halo, nt=9)
    want = [s.integrate(a, 9).clone() for s, a in zip(solvers, x0s)]
    try:
        for tile in (None, (256, 1536), (512, 768), (512, 512), (512, 384)):
            if tile:
                ridc.set_batch_tile(*tile)
            uTs = [torch.empty_like(a) for a in x0s]
            ridc.integrate_batch(solvers, x0s, [9] * count, uTs)
            torch.cuda.synchronize()
            for u, w in zip(uTs, want):
                assert torch.equal(u, w), tile
    finally:
        ridc.tune_clear()
        for s in solvers:
            s.close()


def test_a_refused_tile_changes_nothing(env):
    """A tiling that is refused leaves the handle on the kernel it had: a small system, untouched or set
    to the whole range, still runs its steps in one workgroup."""
    torch, ridc = env
    ridc.tune_clear()
    x = workloads.grid_points("periodic", 256, 2 * math.pi)
    x0 = torch.tensor(np.sin(x), dtype=torch.float64, device="cuda")
    prob = dict(dim=1, bc="periodic", n=256, length=2 * math.pi, fe="advect", a=0.01, nu=1e-4, T=0.02,
                nt=400, order=2)
    times = []
    for tiles in (((256, 0, 0),), (), ((512, 0, 2),)):
        s = ridc.Ridc(prob)
        for t in tiles:
            s.set_tile(*t)
        if len(times):
            for bad in ((256, 16, 0), (96, 0, 0), (256, 512, 0)):     # too fine, no such count, too long
                with pytest.raises(ridc.RidcError) as e:
                    s.set_tile(*bad)
                assert e.value.code == ridc.RIDC_E_INVAL
        s.begin(x0, 400)
        ridc.advance([s], 20)
        times.append(s.kernel_time(100)[0])
        s.close()
    _say(f"case: launches per step {times[0]:.2f} us, after refused tiles {times[1]:.2f} and {times[2]:.2f}")
    assert max(times[1:]) < 0.8 * times[0]
