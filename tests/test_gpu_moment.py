"""The moment state (tau = tau_g = 1, FP64, FP32 and FP16 storage, the library's own choice)
against runs of population steps (fused = "never") and against the oracle.

Both advance the same scheme; they differ in the order of sums and in the
contraction of multiply-adds. Bars as for the fused kernel against single
steps: 1e-13 in FP64 after 18 steps, 2e-6 in FP32 (2e-5 of max|u| for
velocities), 1e-12 against the oracle after 150 steps. Lattices around the
widths where a wavefront's 58 stored columns end, narrower than its halo, and
with one to a few rows.
"""
import numpy as np
import pytest

import workloads
from oracle.oracle import ModelParams, Oracle
from paper_2109_12565_amd import Simulation
from paper_2109_12565_amd._lib import TLB_ENUMERIC, TlbError

from test_gpu_parity import field_errors, pop_errors, posts_case, rel
from test_gpu_step2 import CASES, assert_close_state, droplet_case

pytestmark = pytest.mark.gpu

U_WALL = (-0.01, 0.02)


def make(case, precision, fused="auto", **extra):
    return Simulation(dict(case["params"], **extra), case["rho_a"], case["rho_b"], case["temp"],
                      solid=case.get("solid"), t_bottom=case.get("t_bottom"), precision=precision,
                      launch={"fused": fused})


def bars(precision):
    return (1e-13, 1e-13) if precision == "fp64" else (2e-6, 2e-5)


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("name", sorted(CASES))
@pytest.mark.parametrize("u_wall", [(0.0, 0.0), U_WALL])
def test_moment_steps_match_population_steps(precision, name, u_wall):
    case = CASES[name]()
    print(name, precision, u_wall, flush=True)
    a, b = (make(case, precision, f, u_wall=u_wall) for f in ("auto", "never"))
    assert_close_state(a, b, *bars(precision))   # t = 0
    for n in (9, 1, 2, 6):
        a.step(n)
        b.step(n)
    assert a.t == b.t == 18
    assert_close_state(a, b, *bars(precision))


@pytest.mark.parametrize("lx,ly", [(1, 1), (2, 5), (5, 3), (64, 1), (7, 2), (58, 9), (59, 4), (116, 30),
                                   (117, 7), (175, 13)])
def test_moment_edge_shapes_fp64(lx, ly):
    """Velocities get 1e-11 of max|u|, which is small on these lattices."""
    case = droplet_case(lx, ly, seed=lx + ly)
    a, b = (make(case, "fp64", f) for f in ("auto", "never"))
    for n in (7, 4):
        a.step(n)
        b.step(n)
    assert_close_state(a, b, 1e-13, 1e-11)


def test_moment_state_matches_oracle_with_posts_and_moving_walls():
    case = posts_case()
    sim = make(case, "fp64", u_wall=U_WALL)
    ora = Oracle(ModelParams(**dict(case["params"], u_wall=U_WALL)), case["rho_a"], case["rho_b"],
                 case["temp"], solid=case["solid"], t_bottom=case["t_bottom"])
    sim.step(151)
    ora.step(151)
    errs = field_errors(sim.fields(), ora.fields())
    assert max(errs.values()) <= 1e-12, errs
    perr = pop_errors(sim.populations(), ora.post_collision())
    assert max(perr.values()) <= 1e-12, perr


@pytest.mark.parametrize("name", ["small", "posts"])
def test_new_bottom_temperature_between_steps(name):
    """A new bottom temperature enters the observables, fields and stress of
    the current time at once (its wall links are pulled again), leaves the
    populations, and enters the steps that follow; also twice, and with a
    velocity start at t = 0."""
    case = CASES[name]()
    shape = case["rho_a"].shape
    rng = np.random.default_rng(3)
    u = rng.uniform(-0.02, 0.02, (2,) + shape)
    sims = [Simulation(case["params"], case["rho_a"], case["rho_b"], case["temp"], ux0=u[0], uy0=u[1],
                       solid=case.get("solid"), t_bottom=case["t_bottom"], precision="fp64",
                       launch={"fused": f}) for f in ("auto", "never")]

    def compare():
        got, ref = ((s.fields(), s.observables(), s.stress(), s.populations()) for s in sims)
        errs = field_errors(got[0], ref[0])
        assert max(errs.values()) <= 1e-13, errs
        for k in ref[1]:
            assert got[1][k] == pytest.approx(ref[1][k], rel=1e-12, abs=1e-14), k
        for k in ref[2]:
            assert rel(got[2][k], ref[2][k]) <= 1e-12, k
        assert max(pop_errors(got[3], ref[3]).values()) <= 1e-13

    compare()
    for n in (0, 5, 0, 1):
        for s in sims:
            s.step(n)
        for scale in (1.0, 1.3):
            for s in sims:
                s.set_bottom_temperature(scale * case["t_bottom"])
            compare()
    for s in sims:
        s.step(3)
    compare()


@pytest.mark.parametrize("n,ckpt", [(1, 1), (2, 1), (30, 1), (1, 4), (8, 4), (9, 4), (30, 7)])
def test_taped_moment_run_leaves_the_state_of_plain_steps(n, ckpt):
    """The taped run's state, previous level (stress) and loss are those of
    tlb_step, wherever checkpoints fall; its gradient is that of the
    population run."""
    case = workloads.small()
    a, b, c = make(case, "fp64"), make(case, "fp64"), make(case, "fp64", "never")
    for s in (a, b, c):
        s.step(3)
    loss, ref = a.forward_taped(n, ckpt), c.forward_taped(n, ckpt)
    b.step(n)
    assert np.array_equal(a.populations(), b.populations())
    sa, sb = a.stress(), b.stress()
    for k in sa:
        assert np.array_equal(sa[k], sb[k]), k
    assert loss == pytest.approx(ref, rel=1e-13)
    g, r = a.adjoint(n), c.adjoint(n)
    assert np.abs(g - r).max() <= 1e-11 * np.abs(r).max()
    a.step(2)
    b.step(2)
    assert np.array_equal(a.populations(), b.populations())


def test_moment_state_translates_bitwise():
    """A start shifted by 37 columns gives the shifted result bit for bit: no
    column depends on where its wavefront begins."""
    case = posts_case(lx=150, ly=60, seed=9)
    a = make(case, "fp32")
    sh = lambda z: np.roll(z, 37, axis=-1)
    b = make(dict(params=case["params"], **{k: sh(case[k]) for k in ("rho_a", "rho_b", "temp", "solid", "t_bottom")}),
             "fp32")
    a.step(60)
    b.step(60)
    fa, fb = a.fields(), b.fields()
    for k in fa:
        assert np.array_equal(sh(fa[k]), fb[k]), k


@pytest.mark.parametrize("precision", ["fp32", "fp16dev"])
@pytest.mark.parametrize("name", ["small", "posts", "three_strips_short", "narrow"])
@pytest.mark.parametrize("lanes", [128, 256])
def test_moment_steps_are_the_fused_launches_bit_for_bit(precision, name, lanes):
    """In FP32 arithmetic moment steps evaluate the fused launches' operations one
    by one, the 16-bit rounding of stored populations included: populations and
    fields are the same bits after calls of any length, so a trajectory does not
    depend on which of them took it."""
    case = CASES[name]()
    a = make(case, precision)
    b = Simulation(case["params"], case["rho_a"], case["rho_b"], case["temp"], solid=case.get("solid"),
                   t_bottom=case.get("t_bottom"), precision=precision,
                   launch={"fused": "always", "fused_lanes": lanes})
    for n in (0, 1, 2, 3, 4, 9, 60):
        a.step(n)
        b.step(n)
        assert np.array_equal(a.populations(), b.populations()), (n, a.t)
        fa, fb = a.fields(), b.fields()
        for k in fa:
            assert np.array_equal(fa[k], fb[k]), (n, a.t, k)


@pytest.mark.parametrize("n", [1, 2, 3, 4, 5])
@pytest.mark.parametrize("name", ["small", "posts"])
@pytest.mark.parametrize("precision", ["fp64", "fp32", "fp16dev"])
def test_calls_that_read_the_previous_level(precision, name, n):
    """Stress, row averages and, under a new bottom temperature, observables,
    fields and droplets are formed from M(t-1), whatever the number of steps
    and the form that 16-bit storages left it in. Against the fused launches,
    whose populations are the same bits in FP32 arithmetic: the stress terms
    are at most 10 roundings of values below 1 (1e-6 absolute)."""
    case = CASES[name]()
    sims = [make(case, precision, f, u_wall=U_WALL) for f in ("auto", "always")]
    double = precision == "fp64"

    def compare(where):
        got, ref = ((s.stress(), s.row_averages(), s.observables(), s.fields(), s.droplets(0.8, labels=True))
                    for s in sims)
        for k in ref[0]:
            err = np.abs(got[0][k] - ref[0][k]).max()
            assert err <= (1e-13 if double else 1e-6), (where, k, err)
        for k, bar in (("u_av", 1e-13 if double else 1e-6), ("pxy_av", 1e-13 if double else 1e-6)):
            err = np.abs(got[1][k] - ref[1][k]).max()
            assert err <= bar, (where, k, err)
        for k in ref[2]:
            assert got[2][k] == pytest.approx(ref[2][k], rel=1e-12 if double else 2e-5, abs=1e-13), (where, k)
        errs = field_errors(got[3], ref[3])
        assert max(errs[k] for k in ("rho_a", "rho_b", "temp")) <= bars(precision)[0], (where, errs)
        assert max(errs["ux"], errs["uy"]) <= (1e-12 if double else 2e-5), (where, errs)
        for k in ("root", "size", "label"):
            assert np.array_equal(got[4][k], ref[4][k]), (where, k)

    print(precision, name, n, flush=True)
    for s in sims:
        s.step(n)
    compare("as stepped")
    for s in sims:
        s.set_bottom_temperature(1.3 * case["t_bottom"])
    compare("new bottom temperature")
    for s in sims:
        s.step(0)
    compare("after no step")
    for s in sims:
        s.step(n + 1)
    compare("stepped on")


@pytest.mark.parametrize("precision", ["fp64", "fp32", "fp16dev"])
@pytest.mark.parametrize("lx,ly", [(1, 1), (2, 5), (5, 3), (64, 1), (7, 2), (59, 4), (116, 30), (117, 7)])
def test_stress_on_edge_shapes(precision, lx, ly):
    """Stress and row averages, formed from moments, at the widths where a
    wavefront's columns end and with one to a few rows; t = 0 with a velocity
    start included. Bars as in the test above."""
    case = droplet_case(lx, ly, seed=lx + ly)
    rng = np.random.default_rng(lx)
    u = rng.uniform(-0.02, 0.02, (2, ly, lx))
    bar = 1e-13 if precision == "fp64" else 1e-6
    print(precision, lx, ly, flush=True)
    sims = [Simulation(dict(case["params"], u_wall=U_WALL), case["rho_a"], case["rho_b"], case["temp"], ux0=u[0],
                       uy0=u[1], t_bottom=case["t_bottom"], precision=precision, launch={"fused": f})
            for f in ("auto", "always")]
    for n in (0, 1, 3, 2):
        for s in sims:
            s.step(n)
        got, ref = (dict(s.stress(), **s.row_averages()) for s in sims)
        for k in ref:
            assert np.abs(got[k] - ref[k]).max() <= bar, (n, k)


@pytest.mark.parametrize("precision", ["fp64", "fp32", "fp16dev", "bf16dev", "fix16dev"])
def test_launch_info_tells_what_the_steps_advance(precision):
    case = CASES["small"]()
    print(precision, flush=True)
    info = make(case, precision).launch_info()
    assert (info["moment_rows"] > 0) == (precision in ("fp64", "fp32", "fp16dev"))
    if info["moment_rows"]:
        ly, lx = case["rho_a"].shape
        assert info["moment_strip"] <= 58 and info["moment_strip"] * info["moment_grid_x"] >= lx
        assert info["moment_rows"] * info["moment_grid_y"] >= ly and info["moment_tiles"] == 0
    for fused in ("never", "always"):
        assert make(case, precision, fused).launch_info()["moment_rows"] == 0
    assert make(case, precision, tau=1.2).launch_info()["moment_rows"] == 0
    posts = make(CASES["posts"](), precision).launch_info()
    assert (posts["moment_tiles"] > posts["moment_linked"] > 0) == (posts["moment_rows"] > 0)


def test_launch_info_near_the_4_gib_limit():
    """3.6 and 4.1 GiB of populations on either side of the limit."""
    for ly, moments in ((4400, True), (5000, False)):
        a = np.full((ly, 4096), 0.7)
        print("fp64 4096 x", ly, flush=True)
        with Simulation(dict(CASES["small"]()["params"]), a, a, a, t_bottom=np.ones(4096), precision="fp64") as sim:
            assert (sim.launch_info()["moment_rows"] > 0) == moments


@pytest.mark.parametrize("precision", ["fp32", "fp16dev"])
@pytest.mark.parametrize("name", ["small", "posts", "narrow"])
def test_moving_walls_are_the_fused_launches_bit_for_bit(precision, name):
    case = CASES[name]()
    print(precision, name, flush=True)
    a, b = (make(case, precision, f, u_wall=U_WALL) for f in ("auto", "always"))
    for n in (0, 1, 2, 3, 4, 9, 60):
        a.step(n)
        b.step(n)
        assert np.array_equal(a.populations(), b.populations()), (n, a.t)



@pytest.mark.parametrize("precision", ["fp32", "fp16dev"])
@pytest.mark.parametrize("lx,ly", [(1, 1), (2, 5), (5, 3), (64, 1), (7, 2), (58, 9), (59, 4), (116, 30),
                                   (117, 7), (175, 13)])
def test_moment_edge_shapes_are_the_fused_launches_bit_for_bit(precision, lx, ly):
    case = droplet_case(lx, ly, seed=lx + ly)
    print(precision, lx, ly, flush=True)
    a, b = (make(case, precision, f) for f in ("auto", "always"))
    for n in (7, 4, 1):
        a.step(n)
        b.step(n)
        assert np.array_equal(a.populations(), b.populations()), (n, a.t)


@pytest.mark.parametrize("name", ["small", "posts"])
def test_fp16_moment_run_against_the_oracle(name):
    """The default FP16 path keeps its mass to the rounding of FP32 rest
    populations (2^-24 a node and step, random in sign: 1e-6 of the whole) and
    stays within 16-bit rounding of the double-precision run: deviations below
    2 are stored to 2^-11, the moving populations' share of a density is w <=
    1/9 of that each, so 2e-3 of the largest value after 40 steps is ample."""
    case = CASES[name]()
    print(name, flush=True)
    sim = make(case, "fp16dev")
    ora = Oracle(ModelParams(**case["params"]), case["rho_a"], case["rho_b"], case["temp"],
                 solid=case.get("solid"), t_bottom=case["t_bottom"])
    start = sim.observables()
    sim.step(40)
    ora.step(40)
    end = sim.observables()
    for k in ("mass_a", "mass_b"):
        assert end[k] == pytest.approx(start[k], rel=1e-6)
    f, r = sim.fields(), ora.fields()
    for k in ("rho_a", "rho_b", "temp"):
        assert np.abs(f[k] - r[k]).max() <= 2e-3 * np.abs(r[k]).max(), k


@pytest.mark.parametrize("precision", ["fp64", "fp32", "fp16dev"])
@pytest.mark.parametrize("bad", [np.nan, np.inf])
def test_a_broken_density_spreads_as_in_population_steps(precision, bad):
    """NaN reaches the same nodes, through forces and streaming alike, and the
    observables report it. (FP64 forms a force's x part from differences that
    pass over the node's own column, where a NaN above or below it stays, so
    u_x is NaN at nodes whose u_y alone is NaN otherwise; their populations are
    NaN either way.)"""
    case = dict(posts_case())
    ly, lx = case["rho_a"].shape
    case["rho_a"] = case["rho_a"].copy()
    case["rho_a"][ly // 2, lx // 2] = case["rho_a"][ly - 3, 0] = bad
    print(precision, bad, flush=True)
    sims = [make(case, precision, f) for f in ("auto", "never")]
    for n in (0, 1, 2):
        for s in sims:
            s.step(n)
        got, ref = (s.fields() for s in sims)
        for k in ("rho_a", "rho_b", "temp"):
            assert np.array_equal(np.isnan(got[k]), np.isnan(ref[k])), (n, k)
        u, v = (np.isnan(f["ux"]) | np.isnan(f["uy"]) for f in (got, ref))
        assert np.array_equal(u, v), n
        got, ref = (np.isnan(s.populations()) for s in sims)
        assert np.array_equal(got, ref)
        for s in sims:
            with pytest.raises(TlbError) as e:
                s.observables()
            assert e.value.code == TLB_ENUMERIC
