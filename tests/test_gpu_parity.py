"""GPU parity: the HIP path (through the C ABI) against the FP64 oracle.

Bar: FP64 storage -> max relative density error <= 1e-10 and velocity error
<= 1e-10 (absolute, lattice units) after the stated steps; FP32 deviation
storage -> the per-case tolerance written in the test, derived from FP32
rounding (unit roundoff 6e-8) accumulated over the run.
"""
import numpy as np
import pytest

import lbm_inputs as L
from oracle import oracle as O
from oracle import thermo as T
from tests.gpu_cases import Case, drop_case_inputs, max_rel, run_gpu, run_oracle, slab_case_inputs

pytestmark = pytest.mark.gpu

FP64_RHO_TOL = 1e-10
FP64_U_TOL = 1e-10


def _cmp64(case, rho0, u0, steps):
    r_o, U_o, t_o = run_oracle(case, rho0, u0, steps)
    assert np.all(np.isfinite(r_o)) and np.all(np.isfinite(U_o)), "reference run diverged"
    r_g, U_g, t_g = run_gpu(case, rho0, u0, steps)
    assert np.all(np.isfinite(r_g))
    err_r = max_rel(r_g, r_o)
    err_u = float(np.abs(U_g - U_o).max())
    assert err_r <= FP64_RHO_TOL, f"max rel rho error {err_r:.3e}"
    assert err_u <= FP64_U_TOL, f"max U error {err_u:.3e}"
    assert abs(t_g[0] - t_o[0]) <= 1e-12 * abs(t_o[0])
    return err_r, err_u, t_g


def test_flat_interface_d2q9_64x64_fp64_1000_steps():
    # vdW a = 9/49, b = 2/21 at T/Tc = 0.9, slab in the middle half, tanh width 4, noise 1e-4
    case = Case(2, 64, 64)
    rho0, u0 = slab_case_inputs(case, 4.0, 1e-4, 1001)
    _, _, tot = _cmp64(case, rho0, u0, 1000)
    assert abs(tot[0] - rho0.sum()) <= 1e-13 * rho0.sum()     # exact mass conservation


def test_static_drop_d2q9_ragged_fp64():
    # 100 x 70: two x-tiles with a ragged tail, y not a multiple of the tile height
    case = Case(2, 100, 70, a=0.0225, T_reduced=0.8)
    rho0, u0 = drop_case_inputs(case, 20.0, 4.0, 1e-4, 1002)
    _cmp64(case, rho0, u0, 400)


@pytest.mark.parametrize("eos,a,om,tr,kappa", [(T.VDW, 0.02, 0.0, 0.7, 0.02), (T.PR, 0.005, 0.344, 0.6, 0.02),
                                              (T.RKS, 0.01, 0.344, 0.7, 0.02), (T.CS, 0.005, 0.0, 0.7, 0.02),
                                              (T.SC1, 0.0, 0.0, 0.9, 0.05), (T.SC2, 0.0, 0.0, 0.9, 0.05)])
def test_every_eos_d2q9_fp64(eos, a, om, tr, kappa):
    case = Case(2, 48, 20, eos=eos, a=a, acentric=om, T_reduced=tr, kappa=kappa)
    rho0, u0 = slab_case_inputs(case, 4.0, 1e-4, 7)
    _cmp64(case, rho0, u0, 300)


# force models (Sec. 2.3.4): the single-ring Shan-Chen force (eq SCforce), the dual-range force
# (eq DRforce) and general stencil coefficients, with Shan-Chen and cubic EOS
FORCE_CASES_2D = [(O.FORCE_SHAN_CHEN, (0.0, 0.0, 0.0, 0.0), T.SC1, 0.0, 0.0, 0.9),
                  (O.FORCE_DUAL_RANGE, (1.1, 0.0, 0.0, 0.0), T.VDW, 0.02, 0.0, 0.8),
                  (O.FORCE_GENERAL, (1.2, -0.1, 0.04, -0.02), T.VDW, 0.02, 0.0, 0.8)]


@pytest.mark.parametrize("model,g,eos,a,om,tr", FORCE_CASES_2D)
def test_force_models_d2q9_fp64(model, g, eos, a, om, tr):
    case = Case(2, 48, 20, eos=eos, a=a, acentric=om, T_reduced=tr, kappa=0.0, force_model=model, force_g=g)
    rho0, u0 = slab_case_inputs(case, 4.0, 1e-4, 7)
    _cmp64(case, rho0, u0, 300)


@pytest.mark.parametrize("model,g,eos,a,om,tr", [(O.FORCE_SHAN_CHEN, (0.0, 0.0, 0.0, 0.0), T.SC2, 0.0, 0.0, 0.9),
                                                 (O.FORCE_DUAL_RANGE, (1.2, 0.0, 0.0, 0.0), T.PR, 0.005046, 0.344,
                                                  0.6)])
def test_force_models_d3q27_fused_fp64_and_fp32(model, g, eos, a, om, tr):
    # through the single-pass kernels (x ragged over two tiles): FP64 element by element, and
    # FP32 deviation storage on the densities
    case = Case(3, 70, 24, 20, eos=eos, a=a, acentric=om, T_reduced=tr, kappa=0.0, force_model=model, force_g=g)
    rho0, u0 = drop_case_inputs(case, 6.0, 4.0, 1e-5, 1004, centre=(35.0, 12.0, 10.0))
    _cmp64(case, rho0, u0, 100)
    if eos == T.SC2:
        rv, _ = case.coexistence()
        r32, _, _ = run_gpu(case, rho0, u0, 100, precision=1, rho_ref=rv)
        r64, _, _ = run_oracle(case, rho0, u0, 100)
        assert max_rel(r32, r64) < 1e-4


def test_ideal_gas_shear_wave_fp64():
    case = Case(2, 40, 8, eos=T.IDEAL, kappa=0.0, tau=0.7)
    x = np.tile(np.arange(40), 8).astype(float)
    u0 = np.zeros((2, case.N)); u0[1] = 1e-3 * np.sin(2 * np.pi * x / 40)
    _cmp64(case, np.ones(case.N), u0, 200)


def test_drop_d3q27_periodic_fp64():
    # PR at T/Tc = 0.6 (density ratio 853); 70 x 36 x 20: x ragged over two tiles
    case = Case(3, 70, 36, 20, eos=T.PR, a=0.005046, acentric=0.344, T_reduced=0.6)
    rho0, u0 = drop_case_inputs(case, 8.0, 5.0, 1e-5, 1003, centre=(35.0, 18.0, 10.0))
    _cmp64(case, rho0, u0, 100)


@pytest.mark.parametrize("eos", [T.SC1, T.SC2])
def test_shan_chen_drop_d3q27_fp64_and_fp32(eos):
    # Shan-Chen EOS through the fused D3Q27 kernels: FP64 against the oracle element by
    # element, FP32 deviation storage on the bulk densities
    case = Case(3, 70, 20, 24, eos=eos, T_reduced=0.9, kappa=0.05)
    rho0, u0 = drop_case_inputs(case, 6.0, 3.0, 1e-4, 1004, centre=(35.0, 10.0, 12.0))
    _cmp64(case, rho0, u0, 100)
    rv, _ = case.coexistence()
    r32, _, _ = run_gpu(case, rho0, u0, 100, precision=1, rho_ref=rv)
    r64, _, _ = run_oracle(case, rho0, u0, 100)
    assert max_rel(r32, r64) < 1e-4


def test_textured_wall_d3q27_variable_viscosity_fp64():
    # pillar mask with floor, two viscosities (nu_v = 15 nu_l), moving drop: drop-impact shape at
    # reduced size; T/Tc = 0.6 (at 0.5 this start diverges in the oracle as well)
    nx, ny, nz = 32, 32, 40
    mask = L.pillar_mask(nx, ny, nz, 4, 4, 6)
    a, tr, tau = 0.005046, 0.6, 0.6
    fl = T.Fluid(T.PR, a, 2 / 21, tr, 1.0, 0.344)
    rv, rl, _ = T.coexistence(fl)
    case = Case(3, nx, ny, nz, eos=T.PR, a=a, acentric=0.344, T_reduced=tr, tau=tau,
                tau_vapour=0.5 + 15 * (tau - 0.5), rho_wall=rv, mask=mask)
    rho0 = L.drop(nx, ny, nz, 8.0, rl, rv, 5.0, centre=(16.0, 16.0, 24.0), noise=1e-5, seed=1005)
    u0 = L.impact_drop_velocity(rho0, rl, rv, 3, -0.05, 2)
    _cmp64(case, rho0, u0, 60)


def test_random_mask_d2q9_fp64():
    nx, ny = 37, 29
    mask = L.random_mask(nx, ny, 1, 0.1, 21)
    fl = T.Fluid(T.VDW, 0.02, 2 / 21, 0.8)
    rv, rl, _ = T.coexistence(fl)
    case = Case(2, nx, ny, a=0.02, T_reduced=0.8, rho_wall=0.5 * (rv + rl), mask=mask,
                tau_vapour=0.9)
    rho0, u0 = L.random_state(nx * ny, 2, rv, rl, 0.02, 31)
    _cmp64(case, rho0, u0, 150)


@pytest.mark.parametrize("dims", [(1, 1, 1), (2, 3, 1), (3, 5, 1), (5, 1, 1)])
def test_degenerate_tiny_periodic_d2q9(dims):
    # grids smaller than the two-ring stencil: neighbours wrap onto the node itself
    nx, ny, _ = dims
    case = Case(2, nx, ny, a=0.02, T_reduced=0.8)
    fl = case.fluid()
    rv, rl, _ = T.coexistence(fl)
    rho0, u0 = L.random_state(nx * ny, 2, rv, 0.5 * (rv + rl), 0.02, 41)
    _cmp64(case, rho0, u0, 50)


@pytest.mark.parametrize("dims", [(1, 1, 1), (3, 2, 4), (65, 1, 3)])
def test_degenerate_tiny_periodic_d3q27(dims):
    nx, ny, nz = dims
    case = Case(3, nx, ny, nz, a=0.02, T_reduced=0.8)
    rv, rl, _ = T.coexistence(case.fluid())
    rho0, u0 = L.random_state(nx * ny * nz, 3, rv, 0.5 * (rv + rl), 0.02, 43)
    _cmp64(case, rho0, u0, 30)


def test_init_then_moments_returns_inputs():
    case = Case(3, 20, 12, 9, eos=T.PR, a=0.005046, acentric=0.344, T_reduced=0.6)
    rho0, u0 = L.random_state(case.N, 3, 0.1, 5.0, 0.05, 3)
    r_g, U_g, _ = run_gpu(case, rho0, u0, 0)
    r_o, U_o, _ = run_oracle(case, rho0, u0, 0)
    assert max_rel(r_g, rho0) < 1e-14
    assert np.abs(U_g - U_o).max() < 1e-12


def test_init_with_flow_velocity_round_trips():
    # f = f_eq(rho, U - S/(2 rho)): the moments of the initial state return (rho, U)
    case = Case(3, 30, 20, 12, eos=T.PR, a=0.005046, acentric=0.344, T_reduced=0.6)
    rv, rl = case.coexistence()
    rho0, U0 = L.random_state(case.N, 3, rv, rl, 0.05, 19)
    r_g, U_g, _ = run_gpu(case, rho0, U0, 0)
    assert max_rel(r_g, rho0) < 1e-14
    assert np.abs(U_g - U0).max() < 1e-13


# ---------------------------------------------------------------- FP32 deviation storage
def _bulk(r, nx, ny, nz, xs):
    return float(r.reshape(nz, ny, nx)[:, :, xs].mean())


def test_fp32_dev_flat_interface_error_stated():
    # FP32 storage of f - w rho_ref with rho_ref = rho_v; 1000 steps of the 64x64 flat interface.
    # Stated: coexistence (bulk) densities within 1e-5 relative of the FP64 oracle, pointwise
    # density within 1e-3 (the slab position is a neutral mode, FP32 rounding shifts it slightly),
    # mass drift below 1e-6.
    case = Case(2, 64, 64)
    rho0, u0 = slab_case_inputs(case, 4.0, 1e-4, 1001)
    rv, rl = case.coexistence()
    r_o, U_o, t_o = run_oracle(case, rho0, u0, 1000)
    r_g, U_g, t_g = run_gpu(case, rho0, u0, 1000, precision=1, rho_ref=rv)
    for xs in (slice(28, 36), slice(0, 4)):
        a, b = _bulk(r_g, 64, 64, 1, xs), _bulk(r_o, 64, 64, 1, xs)
        assert abs(a - b) / b < 1e-5, f"bulk density {a} vs {b}"
    assert max_rel(r_g, r_o) < 1e-3
    assert abs(t_g[0] - t_o[0]) / t_o[0] < 1e-6


def test_fp32_dev_drop_d3q27_error_stated():
    # 48^3 PR drop at T/Tc = 0.6 (ratio 853), 200 steps; stated: centre and far-field density
    # within 1e-4 relative of the FP64 oracle, mass drift below 1e-6
    case = Case(3, 48, 48, 48, eos=T.PR, a=0.005046, acentric=0.344, T_reduced=0.6)
    rho0, u0 = drop_case_inputs(case, 12.0, 5.0, 1e-5, 1003)
    rv, rl = case.coexistence()
    r_o, _, t_o = run_oracle(case, rho0, u0, 200)
    assert np.all(np.isfinite(r_o)), "reference run diverged"
    r_g, _, t_g = run_gpu(case, rho0, u0, 200, precision=1, rho_ref=rv)
    c = (slice(22, 26), slice(22, 26), slice(22, 26))
    f = (slice(0, 3), slice(0, 3), slice(0, 3))
    for sl in (c, f):
        a, b = float(r_g.reshape(48, 48, 48)[sl].mean()), float(r_o.reshape(48, 48, 48)[sl].mean())
        assert abs(a - b) / b < 1e-4, f"density {a} vs {b}"
    assert abs(t_g[0] - t_o[0]) / t_o[0] < 1e-6


# ---------------------------------------------------------------- runtime behaviour
def test_checkpoint_resume_bitwise():
    import paper_2112_01975_amd as P
    case = Case(3, 24, 20, 16, eos=T.PR, a=0.005046, acentric=0.344, T_reduced=0.6)
    rho0, u0 = drop_case_inputs(case, 6.0)
    for prec in (0, 1):
        with P.Simulation(case.params(prec, 0.01)) as s:
            s.init(rho0, u0).step(10)
            snap = P.lbm_get_populations(s.ctx)
            s.step(15)
            r1, U1, _ = s.moments()
            P.lbm_set_populations(s.ctx, snap)
            s.step(15)
            r2, U2, _ = s.moments()
        assert np.array_equal(r1, r2) and np.array_equal(U1, U2)


def test_repeat_run_is_bitwise_deterministic():
    case = Case(3, 40, 24, 12, eos=T.PR, a=0.005046, acentric=0.344, T_reduced=0.6)
    rho0, u0 = drop_case_inputs(case, 7.0)
    a = run_gpu(case, rho0, u0, 20, precision=1, rho_ref=0.0102)
    b = run_gpu(case, rho0, u0, 20, precision=1, rho_ref=0.0102)
    assert np.array_equal(a[0], b[0]) and np.array_equal(a[1], b[1]) and np.array_equal(a[2], b[2])


_GRAPH_CASES = {
    2: dict(args=(2, 70, 33), kw=dict(a=0.02, T_reduced=0.8, rho_wall=0.9, mask=L.random_mask(70, 33, 1, 0.04, 11))),
    3: dict(args=(3, 24, 20, 16), kw=dict(eos=T.PR, a=0.005046, acentric=0.344, T_reduced=0.6)),
}


@pytest.mark.parametrize("lattice,two_pass,check_every", [(2, "0", 50), (2, "1", 50), (3, "1", 50), (2, "0", -1)])
@pytest.mark.parametrize("prec", [0, 1])
def test_captured_step_blocks_match_launched_steps_bitwise(lattice, two_pass, check_every, prec, monkeypatch):
    # Steps off the fused D3Q27 kernel (the D2Q9 single pass, the two-pass step of either
    # lattice) replay a captured block of 32 steps. Against the same steps launched one by one
    # (LBM2P_GRAPH=0) the populations agree bit for bit after every call. The calls mix replays
    # from either lattice, plain steps, watchdog checks inside a call (check_every 50), state
    # reads, and a caller stream. Without checks (check_every -1) the first call leaves its
    # plain steps queued when the next call captures its graph.
    import torch

    import paper_2112_01975_amd as P
    monkeypatch.setenv("LBM2P_TWO_PASS", two_pass)
    gc = _GRAPH_CASES[lattice]
    case = Case(*gc["args"], **gc["kw"])
    rv, _ = case.coexistence()
    rho_ref = rv if prec else 0.0
    rho0, u0 = drop_case_inputs(case, min(case.nx, case.ny) / 4)
    sims = {}
    try:
        for g in ("1", "0"):
            monkeypatch.setenv("LBM2P_GRAPH", g)
            sims[g] = P.Simulation(case.params(prec, rho_ref, check_every=check_every)).init(rho0, u0)
        calls = ((5, 70), 64, 33, 200, 1, 96)   # (5, 70): two calls with no read between them
        for n in calls:
            for g in sims:
                for m in (n if isinstance(n, tuple) else (n,)):
                    sims[g].step(m)
            pa, pb = (P.lbm_get_populations(sims[g].ctx) for g in ("1", "0"))
            print(f"{lattice}D prec {prec}: {n} steps, equal {np.array_equal(pa, pb)}", flush=True)
            assert np.array_equal(pa, pb), n
        stream = torch.cuda.Stream()
        for g in sims:
            P.lbm_set_stream(sims[g].ctx, stream.cuda_stream)
            sims[g].step(64)
            P.lbm_set_stream(sims[g].ctx, None)
        ra, Ua, ta = sims["1"].moments()
        rb, Ub, tb = sims["0"].moments()
        assert np.array_equal(ra, rb) and np.array_equal(Ua, Ub) and np.array_equal(ta, tb)
        assert np.all(np.isfinite(ra))
    finally:
        for sim in sims.values():
            sim.close()


@pytest.mark.parametrize("two_pass", ["0", "1"])
def test_steps_captured_by_the_caller_are_launched_one_by_one(two_pass, monkeypatch):
    # On a stream the caller is capturing, lbm_step launches its steps into the caller's graph
    # instead of capturing a graph of its own. The caller's graph of 32 steps, replayed twice
    # with eager steps between (an even number: the graph holds the lattice current at capture),
    # matches a context that stepped eagerly, bit for bit.
    import torch

    import paper_2112_01975_amd as P
    monkeypatch.setenv("LBM2P_TWO_PASS", two_pass)
    case = Case(2, 64, 40, a=0.02, T_reduced=0.8)
    rho0, u0 = drop_case_inputs(case, 10.0)
    cap = P.Simulation(case.params(0, 0.0, check_every=-1)).init(rho0, u0)
    ref = P.Simulation(case.params(0, 0.0, check_every=-1)).init(rho0, u0)
    stream = torch.cuda.Stream()
    try:
        P.lbm_set_stream(cap.ctx, stream.cuda_stream)
        torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=stream):
            P.lbm_step(cap.ctx, 32)
        for rep in range(2):
            with torch.cuda.stream(stream):
                graph.replay()
            stream.synchronize()
            ref.step(32)
            pa, pb = P.lbm_get_populations(cap.ctx), P.lbm_get_populations(ref.ctx)
            print(f"caller graph replay {rep}: equal {np.array_equal(pa, pb)}", flush=True)
            assert np.array_equal(pa, pb), rep
            cap.step(6)
            ref.step(6)
        P.lbm_set_stream(cap.ctx, None)
    finally:
        cap.close()
        ref.close()


def test_watchdog_reports_divergence_and_domain():
    import paper_2112_01975_amd as P
    case = Case(2, 16, 8, a=0.02, T_reduced=0.8)
    rv, rl = case.coexistence()
    with P.Simulation(case.params(0, 0.0, check_every=1)) as s:
        s.init(np.full(case.N, rv))
        snap = P.lbm_get_populations(s.ctx).view(np.float64).copy()
        snap[5] = np.nan
        with pytest.raises(P.LbmError) as ei:
            P.lbm_set_populations(s.ctx, snap.view(np.uint8))
        assert ei.value.code == P.LBM_E_DIVERGED
        with pytest.raises(P.LbmError) as ei:
            s.step(1)                                   # sticky until re-initialised
        assert ei.value.code == P.LBM_E_DIVERGED
        s.init(np.full(case.N, rv)).step(3)             # recovers
    with P.Simulation(case.params()) as s:
        with pytest.raises(P.LbmError) as ei:
            s.init(np.full(case.N, 1.0 / case.b + 1.0))   # b rho >= 1
        assert ei.value.code == P.LBM_E_DOMAIN


@pytest.mark.parametrize("precision", [0, 1])
def test_watchdog_totals_folded_into_the_fused_step(precision, monkeypatch):
    # in FP32 on a grid without mask the single-pass step accumulates the FP64 totals of its
    # input state (one row per work item: ragged x tiles, several z-chunks and launch windows
    # here), so the check after step k describes the state after k - 1 steps; FP64 checks run
    # the moment pass on the state after k steps. Against the oracle's totals of the state
    # described (FP64 to 1e-12; FP32 deviation storage within its rounding)
    import paper_2112_01975_amd as P
    from oracle import oracle as O
    monkeypatch.setenv("LBM2P_FUSED_TZ", "12")
    case = Case(3, 70, 24, 40, eos=T.PR, a=0.005046, acentric=0.344, T_reduced=0.6)
    rv, rl = case.coexistence()
    rho0 = L.drop(70, 24, 40, 7.0, rl, rv, 5.0, centre=(35.0, 12.0, 20.0), noise=1e-5, seed=1009)
    u0 = np.zeros((3, case.N))
    u0[0] = 0.02                                      # a net momentum to check
    orc = O.Oracle(case.oracle_config()).init(rho0, u0)
    ref = [orc.moments()[2]]
    for _ in range(6):
        ref.append(orc.step(1).moments()[2])
    with P.Simulation(case.params(precision, rv if precision else 0.0, check_every=1)) as s:
        s.init(rho0, u0)
        tot, bad, st = P.lbm_last_check(s.ctx)        # the init check: a moment pass on state 0
        assert st == 0 and bad == 0
        for k in range(1, 7):
            s.step(1)
            tot, bad, st = P.lbm_last_check(s.ctx)
            assert st == (k - 1 if precision == 1 else k) and bad == 0
            M, J = ref[st][0], ref[st][1:]
            tol = 1e-12 if precision == 0 else 2e-6
            assert abs(tot[0] / M - 1) < tol, (k, tot[0], M)
            assert np.abs(tot[1:] - J).max() < tol * M, (k, tot[1:], J)


def test_watchdog_folded_domain_count_one_step_late():
    # plain LBGK (ideal EOS, no force) with a strong velocity wave on 8^3: the state after two
    # steps has 128 nodes with rho <= 0 (outside the domain; all |rho| > 0.5), per the oracle.
    # The FP32 fused step's totals describe its input state, so the check after step 3
    # reports exactly those nodes
    import paper_2112_01975_amd as P
    from oracle import oracle as O
    n = 8
    case = Case(3, n, n, n, eos=T.IDEAL, kappa=0.0, tau=0.8)
    z, y, x = np.meshgrid(np.arange(n), np.arange(n), np.arange(n), indexing="ij")
    u0 = np.zeros((3, n ** 3))
    u0[0] = 0.9 * np.sin(2 * np.pi * x.ravel() / n)
    r2 = O.Oracle(case.oracle_config()).init(np.ones(n ** 3), u0).step(2).moments()[0]
    assert int((r2 <= 0).sum()) == 128
    with P.Simulation(case.params(1, 1.0, check_every=1)) as s:
        s.init(np.ones(n ** 3), u0)
        s.step(1)
        s.step(1)                                     # checks state 1: in the domain
        with pytest.raises(P.LbmError) as ei:
            s.step(1)
        assert ei.value.code == P.LBM_E_DOMAIN
        _, bad, st = P.lbm_last_check(s.ctx)
        assert st == 2 and bad == 128


@pytest.mark.parametrize("dims,masked", [((70, 36, 40), False), ((64, 8, 32), False), ((5, 3, 7), False),
                                         ((48, 20, 36), True)])
def test_fused_step_matches_two_pass_fp32(dims, masked, monkeypatch):
    # the single-pass z-march (default for D3Q27 FP32) against the two-pass step, same inputs:
    # ragged x / y tiles, several z-chunks with a ragged last chunk, tiny grids, a solid mask
    nx, ny, nz = dims
    mask = L.pillar_mask(nx, ny, nz, 4, 4, 5) if masked else None
    case = Case(3, nx, ny, nz, eos=T.PR, a=0.005046, acentric=0.344, T_reduced=0.6,
                rho_wall=0.0102306 if masked else 0.0, mask=mask)
    rv, rl = case.coexistence()
    rho0 = L.drop(nx, ny, nz, min(nx, ny, nz) / 4, rl, rv, 5.0, noise=1e-5, seed=1007)
    monkeypatch.setenv("LBM2P_FUSED_TZ", "16")
    fused = run_gpu(case, rho0, None, 30, precision=1, rho_ref=rv)
    monkeypatch.setenv("LBM2P_TWO_PASS", "1")
    two = run_gpu(case, rho0, None, 30, precision=1, rho_ref=rv)
    assert np.all(np.isfinite(fused[0]))
    assert max_rel(fused[0], two[0]) < 1e-5
    assert np.abs(fused[1] - two[1]).max() < 1e-6


@pytest.mark.parametrize("dims,masked", [((70, 36, 40), False), ((5, 3, 7), False), ((48, 20, 36), True)])
def test_fused_step_matches_two_pass_fp64(dims, masked, monkeypatch):
    # the FP64 z-march (queued moments, collided plane pulled again) against the two-pass
    # step on ragged tiles, several z-chunks, tiny grids and a solid mask: same arithmetic
    # up to the order of a few sums, so agreement to rounding
    nx, ny, nz = dims
    mask = L.pillar_mask(nx, ny, nz, 4, 4, 5) if masked else None
    case = Case(3, nx, ny, nz, eos=T.PR, a=0.005046, acentric=0.344, T_reduced=0.6,
                rho_wall=0.0102306 if masked else 0.0, mask=mask, tau_vapour=1.25 if masked else 0.0)
    rv, rl = case.coexistence()
    rho0 = L.drop(nx, ny, nz, min(nx, ny, nz) / 4, rl, rv, 5.0, noise=1e-5, seed=1007)
    monkeypatch.setenv("LBM2P_FUSED_TZ", "16")
    fused = run_gpu(case, rho0, None, 30)
    monkeypatch.setenv("LBM2P_TWO_PASS", "1")
    two = run_gpu(case, rho0, None, 30)
    assert max_rel(fused[0], two[0]) < 1e-12
    assert np.abs(fused[1] - two[1]).max() < 1e-13
    assert abs(fused[2][0] / two[2][0] - 1) < 1e-14


@pytest.mark.parametrize("precision,masked", [(0, False), (1, False), (0, True)])
def test_fused_step_in_several_launch_windows_matches_two_pass(precision, masked, monkeypatch):
    # 256 x 64 x 32 in z-chunks of 2 planes: 4 x 8 x 16 = 512 work items, more than one per CU,
    # so each step is several launches of one item per CU (with a mask, per plane run)
    nx, ny, nz = 256, 64, 32
    mask = L.pillar_mask(nx, ny, nz, 4, 4, 5) if masked else None
    case = Case(3, nx, ny, nz, eos=T.PR, a=0.005046, acentric=0.344, T_reduced=0.6,
                rho_wall=0.0102306 if masked else 0.0, mask=mask)
    rv, rl = case.coexistence()
    rho0 = L.drop(nx, ny, nz, 12.0, rl, rv, 5.0, centre=(100.0, 30.0, 16.0), noise=1e-5, seed=1009)
    rref = rv if precision == 1 else 0.0
    monkeypatch.setenv("LBM2P_FUSED_TZ", "2")
    fused = run_gpu(case, rho0, None, 20, precision=precision, rho_ref=rref)
    monkeypatch.setenv("LBM2P_TWO_PASS", "1")
    two = run_gpu(case, rho0, None, 20, precision=precision, rho_ref=rref)
    if precision == 0:
        assert max_rel(fused[0], two[0]) < 1e-12 and np.abs(fused[1] - two[1]).max() < 1e-13
    else:
        assert max_rel(fused[0], two[0]) < 1e-5 and np.abs(fused[1] - two[1]).max() < 1e-6


@pytest.mark.parametrize("precision", [0, 1])
def test_fused_step_plane_runs_match_two_pass(precision, monkeypatch):
    # solids in two separate z-bands (a slab at z = 30..31 and scattered nodes at z = 5):
    # the step becomes alternating runs of masked and unmasked launches, with ragged
    # chunks inside the runs; it must agree with the two-pass step as the single-launch
    # fused step does
    nx, ny, nz = 40, 20, 64
    m = np.zeros((nz, ny, nx), np.uint8)
    m[30:32] = 1
    m[30:32, 5:9, 10:14] = 0                       # a hole through the slab
    m[5, 3, 7] = m[5, 12, 30] = 1
    case = Case(3, nx, ny, nz, eos=T.PR, a=0.005046, acentric=0.344, T_reduced=0.6, rho_wall=0.0102306,
                mask=m.ravel())
    rv, rl = case.coexistence()
    rho0 = L.drop(nx, ny, nz, 8.0, rl, rv, 5.0, centre=(20.0, 10.0, 16.0), noise=1e-5, seed=1011)
    rho0 = np.where(m.ravel().astype(bool), rv, rho0)
    rr = rv if precision else 0.0
    monkeypatch.setenv("LBM2P_FUSED_TZ", "10")
    fused = run_gpu(case, rho0, None, 30, precision=precision, rho_ref=rr)
    monkeypatch.setenv("LBM2P_TWO_PASS", "1")
    two = run_gpu(case, rho0, None, 30, precision=precision, rho_ref=rr)
    assert np.all(np.isfinite(fused[0]))
    if precision == 0:
        assert max_rel(fused[0], two[0]) < 1e-12 and np.abs(fused[1] - two[1]).max() < 1e-13
    else:
        assert max_rel(fused[0], two[0]) < 1e-5 and np.abs(fused[1] - two[1]).max() < 1e-6


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("solid_planes", [(0,), (62,), (1, 33)])
def test_fused_plane_run_across_the_periodic_boundary_matches_two_pass(solid_planes, precision, monkeypatch):
    # the planes near a solid at either end of z form one run that wraps (from nz - 3 to 3 for a
    # floor at 0), in z-chunks of a few planes; one chunk then holds planes on both sides of z = 0
    nx, ny, nz = 40, 20, 64
    m = np.zeros((nz, ny, nx), np.uint8)
    for z in solid_planes:
        m[z, :, ::2] = 1
    case = Case(3, nx, ny, nz, eos=T.PR, a=0.005046, acentric=0.344, T_reduced=0.6, rho_wall=0.0102306,
                mask=m.ravel())
    rv, rl = case.coexistence()
    rho0 = L.drop(nx, ny, nz, 8.0, rl, rv, 5.0, centre=(20.0, 10.0, 48.0), noise=1e-5, seed=1012)
    rho0 = np.where(m.ravel().astype(bool), rv, rho0)
    rr = rv if precision else 0.0
    fused = run_gpu(case, rho0, None, 30, precision=precision, rho_ref=rr)
    monkeypatch.setenv("LBM2P_FUSED_TZ", "5")
    ragged = run_gpu(case, rho0, None, 30, precision=precision, rho_ref=rr)
    monkeypatch.setenv("LBM2P_TWO_PASS", "1")
    two = run_gpu(case, rho0, None, 30, precision=precision, rho_ref=rr)
    tol, utol = (1e-12, 1e-13) if precision == 0 else (1e-5, 1e-6)
    for r, u, _ in (fused, ragged):
        assert np.all(np.isfinite(r))
        assert max_rel(r, two[0]) < tol and np.abs(u - two[1]).max() < utol


@pytest.mark.parametrize("masked", [False, True])
@pytest.mark.parametrize("dims", [(64, 4, 4), (66, 5, 9), (130, 61, 37), (130, 61, 1)])
def test_output_fields_at_tile_and_chunk_edges_match_the_oracle(dims, masked):
    # density and velocity of a moving state: one tile, ragged tiles, padded rows (66, 130), and
    # z-chunks of the velocity pass that do not divide nz; FP64, so within the parity bound 1e-10
    D = 2 if dims[2] == 1 else 3
    N = dims[0] * dims[1] * dims[2]
    mask = L.random_mask(*dims, 0.1, 11) if masked else None
    case = Case(D, *dims, a=0.02, T_reduced=0.8, rho_wall=2.0, mask=mask)
    rho0, u0 = L.random_state(N, D, 1.0, 1.3, 0.02, 5)
    for steps in (0, 2):
        r_o, U_o, _ = run_oracle(case, rho0, u0, steps)
        r_g, U_g, _ = run_gpu(case, rho0, u0, steps)
        assert max_rel(r_g, r_o) < 1e-10 and np.abs(U_g - U_o).max() < 1e-10


@pytest.mark.parametrize("dims", [(150, 20, 24), (33, 17, 9), (96, 96, 32), (32, 16, 4)])
def test_fused_tiles_of_32x16_agree_bit_for_bit(dims, monkeypatch):
    # the tile shape changes which thread computes a node, not its arithmetic: FP32 populations of
    # 32 x 16 and 64 x 8 tiles are the same bits, on grids the tiles divide and do not, with the
    # z-chunks of a few planes that small boxes take and with one chunk
    import paper_2112_01975_amd as P
    nx, ny, nz = dims
    case = Case(3, nx, ny, nz, eos=T.PR, a=0.005046, acentric=0.344, T_reduced=0.6)
    rv, rl = case.coexistence()
    rho0 = L.drop(nx, ny, nz, min(dims) / 4, rl, rv, 5.0, noise=1e-5, seed=1013)
    pops = []
    for tx, ty, tz in ((64, 8, 320), (64, 8, 4), (32, 16, 4), (32, 16, 320)):
        monkeypatch.setenv("LBM2P_FUSED_TX", str(tx))
        monkeypatch.setenv("LBM2P_FUSED_TY", str(ty))
        monkeypatch.setenv("LBM2P_FUSED_TZ", str(tz))
        with P.Simulation(case.params(1, rv)) as s:
            s.init(rho0).step(12)
            pops.append(P.lbm_get_populations(s.ctx))
    for p in pops[1:]:
        assert np.array_equal(pops[0], p)


# ---------------------------------------------------------------- batched sweep
def _sweep_cases(n, steps_len_lo=32, steps_len_hi=96):
    """A reduced temperature sweep: D2Q9 4 x L flat interfaces, FP64 from T/Tc >= 0.95."""
    sweep = L.temperature_sweep(n, 0.55, 0.99, steps_len_lo, steps_len_hi, 4)
    fl0 = T.Fluid(T.VDW, 9 / 49, 2 / 21, 0.55)
    a = 9 / 49 * 0.02 / T.kappa_for_width(fl0, 4.0)
    out = []
    for sc in sweep:
        case = Case(2, sc.nx, sc.ny, a=a, T_reduced=sc.T_reduced)
        rv, rl = case.coexistence()
        W = max(4.0, T.interface_width(case.fluid(), 0.02))
        rho0 = L.flat_slab(sc.nx, sc.ny, 1, rl, rv, W, noise=1e-4, seed=2000 + sc.index)
        out.append((sc, case, rho0, rv))
    return out


@pytest.mark.parametrize("stepped", ["1", "0"])
def test_batched_sweep_matches_single_runs_and_oracle(stepped, monkeypatch):
    # both designs: the stepped kernels over every case (default) and one workgroup per case
    monkeypatch.setenv("LBM2P_BATCH_STEPPED", stepped)
    import paper_2112_01975_amd as P
    cases = _sweep_cases(10)
    plist = [c.params(1 if not sc.fp64 else 0, rv if not sc.fp64 else 0.0) for sc, c, _, rv in cases]
    b = P.lbm_batch_create(plist)
    try:
        for i, (sc, c, rho0, rv) in enumerate(cases):
            P.lbm_batch_init_fields(b, i, rho0)
        P.lbm_batch_step(b, 301)          # odd: exercises the lattice parity flip after the graph chunks
        for i, (sc, c, rho0, rv) in enumerate(cases):
            rb, Ub, tb = P.lbm_batch_moments(b, i, c.N, 2)
            rs, Us, ts = run_gpu(c, rho0, None, 301, precision=1 if not sc.fp64 else 0,
                                 rho_ref=rv if not sc.fp64 else 0.0)
            tol = 1e-12 if sc.fp64 else 2e-5
            assert max_rel(rb, rs) < tol, (i, max_rel(rb, rs))
            ro, Uo, to = run_oracle(c, rho0, None, 301)
            if sc.fp64:
                assert max_rel(rb, ro) < FP64_RHO_TOL
                assert np.abs(Ub - Uo).max() < FP64_U_TOL
            else:
                # FP32 deviation storage against the FP64 oracle, node by node: stated bound
                # 1e-4 in density (the FP32 bound of the coexistence densities) and 1e-5 in U
                assert max_rel(rb, ro) < 1e-4, (i, max_rel(rb, ro))
                assert np.abs(Ub - Uo).max() < 1e-5, (i, np.abs(Ub - Uo).max())
    finally:
        P.lbm_batch_destroy(b)


@pytest.mark.parametrize("stepped", ["1", "0"])
def test_batched_mixed_lattices_and_masks(stepped, monkeypatch):
    monkeypatch.setenv("LBM2P_BATCH_STEPPED", stepped)
    import paper_2112_01975_amd as P
    c2 = Case(2, 40, 30, a=0.02, T_reduced=0.8, rho_wall=0.9, mask=L.random_mask(40, 30, 1, 0.05, 3))
    c3 = Case(3, 20, 18, 16, eos=T.PR, a=0.005046, acentric=0.344, T_reduced=0.6)
    rv2, rl2 = c2.coexistence()
    rv3, rl3 = c3.coexistence()
    r2 = L.drop(40, 30, 1, 8.0, rl2, rv2, 4.0, noise=1e-4, seed=5)
    r3 = L.drop(20, 18, 16, 5.0, rl3, rv3, 5.0, noise=1e-5, seed=6)
    b = P.lbm_batch_create([c2.params(0), c3.params(0)])
    try:
        P.lbm_batch_init_fields(b, 0, r2)
        P.lbm_batch_init_fields(b, 1, r3)
        P.lbm_batch_step(b, 60)
        for i, (c, r0) in enumerate(((c2, r2), (c3, r3))):
            rb, Ub, _ = P.lbm_batch_moments(b, i, c.N, c.lattice)
            ro, Uo, _ = run_oracle(c, r0, None, 60)
            assert max_rel(rb, ro) < FP64_RHO_TOL
            assert np.abs(Ub - Uo).max() < FP64_U_TOL
    finally:
        P.lbm_batch_destroy(b)


@pytest.mark.parametrize("stepped", ["1", "0"])
def test_batched_force_models(stepped, monkeypatch):
    # cases with different force models side by side in one batch: each against the oracle
    # (FP64) and against its single run (bit for bit)
    monkeypatch.setenv("LBM2P_BATCH_STEPPED", stepped)
    import paper_2112_01975_amd as P
    cases = [Case(2, 48, 20, eos=eos, a=a, acentric=om, T_reduced=tr, kappa=0.0, force_model=model, force_g=g)
             for model, g, eos, a, om, tr in FORCE_CASES_2D]
    cases.append(Case(2, 48, 20, a=0.02, T_reduced=0.8))          # the default Korteweg force
    inits = [slab_case_inputs(c, 4.0, 1e-4, 7)[0] for c in cases]
    b = P.lbm_batch_create([c.params(0) for c in cases])
    try:
        for i, r0 in enumerate(inits):
            P.lbm_batch_init_fields(b, i, r0)
        P.lbm_batch_step(b, 120)
        for i, (c, r0) in enumerate(zip(cases, inits)):
            rb, Ub, _ = P.lbm_batch_moments(b, i, c.N, 2)
            ro, Uo, _ = run_oracle(c, r0, None, 120)
            assert max_rel(rb, ro) < FP64_RHO_TOL and np.abs(Ub - Uo).max() < FP64_U_TOL, i
            rs, Us, _ = run_gpu(c, r0, None, 120)
            assert max_rel(rb, rs) < 1e-12, i
    finally:
        P.lbm_batch_destroy(b)


def test_batch_block_splits_agree_bit_for_bit_and_tuning_is_cached(monkeypatch, tmp_path):
    # the stepped design's block split (threads per block, nodes per thread) only moves nodes
    # between threads: forced splits give the same bits; the tuner's choice is appended once to
    # the cache file (keyed by GPU target and case list) and read back by the next batch
    import paper_2112_01975_amd as P
    monkeypatch.setenv("LBM2P_BATCH_CHUNK", "16")
    cases = _sweep_cases(6)
    plist = [c.params(1 if not sc.fp64 else 0, rv if not sc.fp64 else 0.0) for sc, c, _, rv in cases]

    def run():
        b = P.lbm_batch_create(plist)
        try:
            for i, (sc, c, rho0, rv) in enumerate(cases):
                P.lbm_batch_init_fields(b, i, rho0)
            P.lbm_batch_step(b, 37)
            return [P.lbm_batch_moments(b, i, c.N, 2)[:2] for i, (sc, c, _, _) in enumerate(cases)]
        finally:
            P.lbm_batch_destroy(b)

    out = {}
    for split in ("256,1", "64,1", "128,2", "64,4"):
        monkeypatch.setenv("LBM2P_BATCH_SPLIT", split)
        out[split] = run()
    for split in ("64,1", "128,2", "64,4"):
        for (ra, Ua), (rb, Ub) in zip(out["256,1"], out[split]):
            assert np.array_equal(ra, rb) and np.array_equal(Ua, Ub), split
    monkeypatch.delenv("LBM2P_BATCH_SPLIT")
    cache = tmp_path / "tune.txt"
    monkeypatch.setenv("LBM2P_TUNE_CACHE", str(cache))
    tuned = run()
    lines = cache.read_text().splitlines()
    assert len(lines) == 1 and lines[0].split()[0].startswith("gfx") and lines[0].split()[2] == "s"
    again = run()
    assert cache.read_text().splitlines() == lines          # read back, not tuned again
    for (ra, Ua), (rb, Ub), (rc, Uc) in zip(out["256,1"], tuned, again):
        assert np.array_equal(ra, rb) and np.array_equal(ra, rc) and np.array_equal(Ua, Uc)


def test_batch_tiles_of_several_steps_agree_bit_for_bit(monkeypatch):
    # D2Q9 cases whose tile fits in LDS advance several steps per launch (tiles with a halo of
    # three columns per step, recomputed by the neighbours); the same per-node functions run
    # in LDS, so every tiling matches the stepped kernels bit for bit: FP32 and FP64 sweep cases,
    # a masked FP64 channel (bounce-back and wall density inside the tile), a D3Q27 case that
    # stays with the stepped kernels, 37 steps (graph chunks of 16 and a remainder, odd tile
    # launches), and tiles wider than some cases
    import paper_2112_01975_amd as P
    monkeypatch.setenv("LBM2P_BATCH_CHUNK", "16")
    sweep = _sweep_cases(5)
    fl = T.Fluid(T.VDW, 0.02, 2 / 21, 0.8)
    rv8, rl8, _ = T.coexistence(fl)
    mask = np.zeros((5, 96), np.uint8)
    mask[0] = 1
    mask[4, 10:40] = 1
    cm = Case(2, 96, 5, a=0.02, T_reduced=0.8, rho_wall=0.5 * (rv8 + rl8), mask=mask.ravel(), accel=(1e-5, 0.0, 0.0))
    c3 = Case(3, 20, 18, 16, eos=T.PR, a=0.005046, acentric=0.344, T_reduced=0.6)
    rv3, rl3 = c3.coexistence()
    cases = [c for _, c, _, _ in sweep] + [cm, c3]
    inits = [r0 for _, _, r0, _ in sweep] + [L.random_state(cm.N, 2, rv8, rl8, 0.02, 77)[0],
                                             L.drop(20, 18, 16, 5.0, rl3, rv3, 5.0, noise=1e-5, seed=6)]
    plist = [c.params(1 if not sc.fp64 else 0, rv if not sc.fp64 else 0.0) for sc, c, _, rv in sweep]
    plist += [cm.params(0), c3.params(1, rv3)]

    def run(tile):
        monkeypatch.setenv("LBM2P_BATCH_TILE", tile)
        b = P.lbm_batch_create(plist)
        try:
            for i, r0 in enumerate(inits):
                P.lbm_batch_init_fields(b, i, r0)
            P.lbm_batch_step(b, 37)
            return [P.lbm_batch_moments(b, i, c.N, c.lattice)[:2] for i, c in enumerate(cases)]
        finally:
            P.lbm_batch_destroy(b)

    ref = run("0,64")
    for tile in ("4,32", "3,64", "4,96", "8,32", "16,128", "4,192", "4,128,128", "5,256,128", "12,384,128"):
        got = run(tile)
        for i, ((ra, Ua), (rb, Ub)) in enumerate(zip(ref, got)):
            assert np.array_equal(ra, rb) and np.array_equal(Ua, Ub), (tile, i)
    # and the masked channel against the oracle (FP64)
    ro, Uo, _ = run_oracle(cm, inits[-2], None, 37)
    assert max_rel(ref[-2][0], ro) < FP64_RHO_TOL and np.abs(ref[-2][1] - Uo).max() < FP64_U_TOL


def test_batch_designs_agree_bit_for_bit(monkeypatch):
    # the stepped kernels and the persistent design run the same per-node device functions in
    # the same order, so every field agrees exactly: FP64 and FP32 cases, both lattices, a mask,
    # an odd step count (a parity flip) split across a graph chunk and a remainder
    import paper_2112_01975_amd as P
    monkeypatch.setenv("LBM2P_BATCH_CHUNK", "16")
    c2 = Case(2, 40, 30, a=0.02, T_reduced=0.8, rho_wall=0.9, mask=L.random_mask(40, 30, 1, 0.05, 3))
    c2b = Case(2, 64, 16, a=0.02, T_reduced=0.8)
    c3 = Case(3, 20, 18, 16, eos=T.PR, a=0.005046, acentric=0.344, T_reduced=0.6)
    rv2, rl2 = c2.coexistence()
    rv3, rl3 = c3.coexistence()
    inits = [L.drop(40, 30, 1, 8.0, rl2, rv2, 4.0, noise=1e-4, seed=5),
             L.flat_slab(64, 16, 1, rl2, rv2, 4.0, noise=1e-4, seed=7),
             L.drop(20, 18, 16, 5.0, rl3, rv3, 5.0, noise=1e-5, seed=6)]
    plist = [c2.params(0), c2b.params(1, rv2), c3.params(1, rv3)]
    out = {}
    for stepped in ("1", "0"):
        monkeypatch.setenv("LBM2P_BATCH_STEPPED", stepped)
        b = P.lbm_batch_create(plist)
        try:
            for i, r0 in enumerate(inits):
                P.lbm_batch_init_fields(b, i, r0)
            P.lbm_batch_step(b, 37)
            out[stepped] = [P.lbm_batch_moments(b, i, c.N, c.lattice)[:2] for i, c in enumerate((c2, c2b, c3))]
        finally:
            P.lbm_batch_destroy(b)
    for (ra, Ua), (rb, Ub) in zip(out["1"], out["0"]):
        assert np.array_equal(ra, rb) and np.array_equal(Ua, Ub)


# ------------------------------------------------------------------ body force, per-node wall densities
def _layered_channel(lattice, nx, H, g, tau=1.0, tr=0.77, nz=1):
    """vdW liquid below / vapour above between two-row walls (normal to y for D2Q9, to z
    for D3Q27) whose virtual densities match the adjacent phase; gravity along x."""
    fl0 = T.Fluid(T.VDW, 9 / 49, 2 / 21, tr)
    a = 9 / 49 * 0.02 / T.kappa_for_width(fl0, 4.0)
    rv, rl, _ = T.coexistence(T.Fluid(T.VDW, a, 2 / 21, tr))
    nw = H + 4
    if lattice == 2:
        shape, ny = (nw, nx), nw
        col = np.arange(nw)[:, None] * np.ones((1, nx))
    else:
        shape, ny = (nw, nz, nx), nz
        col = np.arange(nw)[:, None, None] * np.ones((1, nz, nx))
    mask = ((col < 2) | (col >= nw - 2)).astype(np.uint8).ravel()
    wall = np.where(col < nw // 2, rl, rv).ravel()
    rho0 = (0.5 * (rl + rv) - 0.5 * (rl - rv) * np.tanh(2 * (col - 1.5 - H / 2) / 4.0)).ravel()
    if lattice == 2:
        case = Case(2, nx, nw, 1, eos=T.VDW, a=a, T_reduced=tr, kappa=0.02, tau=tau, rho_wall=rv, mask=mask,
                    accel=(g, 0.0, 0.0), rho_wall_field=wall)
    else:   # channel across z: D3Q27 grid (nx, ny = nz_arg, nz = H + 4)
        case = Case(3, nx, ny, nw, eos=T.VDW, a=a, T_reduced=tr, kappa=0.02, tau=tau, rho_wall=rv, mask=mask,
                    accel=(g, 0.0, 0.0), rho_wall_field=wall)
    return case, rho0, (rv, rl)


def test_layered_channel_body_force_d2q9_fp64_and_fp32():
    case, rho0, (rv, rl) = _layered_channel(2, 5, 50, 1e-6)
    _cmp64(case, rho0, None, 3000)
    r32, U32, _ = run_gpu(case, rho0, None, 3000, precision=1, rho_ref=rv)
    r64, U64, _ = run_oracle(case, rho0, None, 3000)
    fl = ~case.mask.astype(bool)
    assert max_rel(r32[fl], r64[fl]) < 1e-4
    assert np.abs(U32 - U64).max() < 1e-3 * np.abs(U64).max()


def test_wall_bounded_channel_body_force_d3q27_fused_fp64_and_fp32():
    # walls across z: the masked fused kernels (plane flags pick the bounce-back planes)
    case, rho0, (rv, rl) = _layered_channel(3, 70, 36, 1e-6, nz=9)
    _cmp64(case, rho0, None, 400)
    r32, U32, _ = run_gpu(case, rho0, None, 400, precision=1, rho_ref=rv)
    r64, U64, _ = run_oracle(case, rho0, None, 400)
    fl = ~case.mask.astype(bool)
    assert max_rel(r32[fl], r64[fl]) < 1e-4
    assert np.abs(U32 - U64).max() < 2e-3 * np.abs(U64).max()


def test_batched_sweep_with_body_force_and_wall_field():
    # the batch kernel's source and wall densities: a layered channel (D2Q9) and a 3D
    # wall-bounded channel in one launch, each against the oracle
    import paper_2112_01975_amd as P
    c2, r2, _ = _layered_channel(2, 5, 40, 2e-6)
    c3, r3, _ = _layered_channel(3, 6, 20, 2e-6, nz=5)
    b = P.lbm_batch_create([c2.params(0), c3.params(0)])
    try:
        P.lbm_batch_init_fields(b, 0, r2)
        P.lbm_batch_init_fields(b, 1, r3)
        P.lbm_batch_step(b, 300)
        for i, (c, r0) in enumerate(((c2, r2), (c3, r3))):
            rb, Ub, _ = P.lbm_batch_moments(b, i, c.N, c.lattice)
            ro, Uo, _ = run_oracle(c, r0, None, 300)
            assert max_rel(rb, ro) < FP64_RHO_TOL
            assert np.abs(Ub - Uo).max() < FP64_U_TOL
            assert np.abs(Uo[0]).max() > 1e-5        # the body force has driven a flow
    finally:
        P.lbm_batch_destroy(b)



# ---------------------------------------------------------------- pitched rows
@pytest.mark.parametrize("dims,masked", [((37, 29, 1), True), ((45, 11, 13), True), ((70, 9, 12), False)])
def test_padded_rows_match_the_oracle(dims, masked, monkeypatch):
    # rows padded to a multiple of 32 nodes (forced for every nx; by default from nx = 64):
    # the step, the initial state, the moments and the checkpoint layout are unchanged
    import paper_2112_01975_amd as P
    monkeypatch.setenv("LBM2P_PITCH_ALL", "1")
    nx, ny, nz = dims
    D = 2 if nz == 1 else 3
    mask = L.random_mask(nx, ny, nz, 0.1, 23) if masked else None
    fl = T.Fluid(T.VDW, 0.02, 2 / 21, 0.8)
    rv, rl, _ = T.coexistence(fl)
    wf = np.random.default_rng(4).uniform(rv, rl, nx * ny * nz) if masked else None
    case = Case(D, nx, ny, nz, a=0.02, T_reduced=0.8, rho_wall=0.5 * (rv + rl), mask=mask, rho_wall_field=wf,
                accel=(1e-5, 0.0, 0.0))
    rho0, u0 = L.random_state(nx * ny * nz, D, rv, rl, 0.02, 37)
    _cmp64(case, rho0, u0, 60)
    with P.Simulation(case.params()) as s:          # checkpoint round trip through the padded layout
        s.init(rho0, u0).step(5)
        snap = P.lbm_get_populations(s.ctx)
        assert snap.size == P.lbm_population_bytes(s.ctx) == (27 if D == 3 else 9) * nx * ny * nz * 8
        s.step(7)
        r1, _, _ = s.moments()
        P.lbm_set_populations(s.ctx, snap)
        s.step(7)
        r2, _, _ = s.moments()
    assert np.array_equal(r1, r2)


def test_batch_step_reports_the_diverged_case():
    # a D2Q9 case started far from equilibrium at tau 0.51 with densities up to b rho = 0.97
    # leaves the EOS domain and turns non-finite within a few steps (the oracle does within 15);
    # the end-of-call check of lbm_batch_step names it, and a sane case beside it does not matter
    import paper_2112_01975_amd as P
    good = Case(2, 48, 4, a=0.02, T_reduced=0.8)
    wild = Case(2, 32, 4, a=0.02, T_reduced=0.8, tau=0.51)
    rv, rl = good.coexistence()
    rng = np.random.default_rng(5)
    b = P.lbm_batch_create([good.params(1, rv), wild.params(0)])
    try:
        P.lbm_batch_init_fields(b, 0, L.flat_slab(48, 4, 1, rl, rv, 4.0, noise=1e-4, seed=9))
        P.lbm_batch_init_fields(b, 1, rng.uniform(0.2, 10.2, wild.N))
        with pytest.raises(P.LbmError) as ei:
            P.lbm_batch_step(b, 60)
        assert ei.value.code == P.LBM_E_DIVERGED and "case 1" in str(ei.value), str(ei.value)
    finally:
        P.lbm_batch_destroy(b)


def test_small_grids_take_the_two_pass_step_by_default(monkeypatch):
    # By default a D3Q27 grid takes the single-pass step only when 16-plane z-chunks of its 64x8
    # tiles give at least one work item per CU: 64^3 gives 32 (two-pass), 128^3 gives 256
    # (single-pass). The default step at 64^3 matches the oracle (FP64, 20 steps).
    import paper_2112_01975_amd as P
    monkeypatch.delenv("LBM2P_FUSED", raising=False)
    for n, single_pass in ((64, False), (128, True)):
        case = Case(3, n, n, n, eos=T.PR, a=0.005046, acentric=0.344, T_reduced=0.6)
        rv, rl = case.coexistence()
        rho0 = L.drop(n, n, n, n / 4, rl, rv, 5.0, noise=1e-5, seed=7)
        with P.Simulation(case.params(0)) as s:
            s.init(rho0)
            _, nl = P.lbm_step_timed(s.ctx, 20)
            assert (nl[0] == 0) == single_pass, (n, list(nl))
            if n == 64:
                r_g, U_g, _ = s.moments()
                r_o, U_o, _ = run_oracle(case, rho0, None, 20)
                assert max_rel(r_g, r_o) <= FP64_RHO_TOL and np.abs(U_g - U_o).max() <= FP64_U_TOL


# the step a box without walls takes by itself (FP64, FP32): cubes around the line, boxes whose rows
# leave most lanes of the two passes' tiles idle, flat ones; and its state against the two-pass step
@pytest.mark.parametrize("dims,single_pass", [((64, 64, 64), (False, False)), ((80, 80, 80), (True, False)), ((96, 96, 96), (True, True)),
                                              ((150, 141, 130), (True, True)), ((8, 300, 300), (True, True)), ((16, 16, 4096), (True, True)),
                                              ((33, 129, 257), (True, True)), ((512, 512, 1), (False, False))])
def test_default_step_of_plain_boxes(dims, single_pass, monkeypatch):
    import paper_2112_01975_amd as P
    monkeypatch.delenv("LBM2P_FUSED", raising=False)
    case = Case(3, *dims, a=0.02, T_reduced=0.8)
    rho0, u0 = L.random_state(case.N, 3, 1.0, 1.3, 0.02, 51)
    for prec in (0, 1):
        got = []
        for two_pass in ("0", "1"):
            monkeypatch.setenv("LBM2P_TWO_PASS", two_pass)
            with P.Simulation(case.params(prec, 1.0 if prec else 0.0)) as s:
                s.init(rho0, u0)
                _, nl = P.lbm_step_timed(s.ctx, 3)
                assert (nl[0] == 0) == (single_pass[prec] and two_pass == "0"), (dims, prec, list(nl))
                got.append(s.moments())
        tol, utol = (1e-12, 1e-12) if prec == 0 else (1e-5, 1e-6)   # bounds of the two-pass comparisons above
        assert max_rel(got[0][0], got[1][0]) < tol and np.abs(got[0][1] - got[1][1]).max() < utol


# chunks of one, two and three planes of the velocity pass, the last chunk ragged
@pytest.mark.parametrize("masked", [False, True])
@pytest.mark.parametrize("dims", [(70, 30, 7), (130, 61, 15), (130, 61, 25)])
def test_output_fields_in_short_marches_match_the_oracle(dims, masked):
    N = dims[0] * dims[1] * dims[2]
    mask = L.random_mask(*dims, 0.1, 12) if masked else None
    case = Case(3, *dims, a=0.02, T_reduced=0.8, rho_wall=2.0, mask=mask)
    rho0, u0 = L.random_state(N, 3, 1.0, 1.3, 0.02, 6)
    r_o, U_o, _ = run_oracle(case, rho0, u0, 1)
    r_g, U_g, _ = run_gpu(case, rho0, u0, 1)
    assert max_rel(r_g, r_o) < 1e-10 and np.abs(U_g - U_o).max() < 1e-10   # the parity bound
