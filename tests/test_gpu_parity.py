"""GPU parity: the HIP path through the C ABI against the FP64 oracle on the
same seeded inputs.  Bar: relative L2 <= 1e-12 per field in FP64, <= 1e-5 in
FP32-mixed (the FP32 run starts from the FP64 input rounded to FP32).  Step
tests also compare the change of every field over the run, x - x(0), whose
bar (tests/fp32_bounds.py) is 1e-5 plus what rounding the stored state costs;
the states here change enough that the bar is close to 1e-5, so a field that
is never updated fails."""
import numpy as np
import pytest

from paper_2502_14148_amd import inputs
from paper_2502_14148_amd.inputs import Physics
from oracle import fv, tendencies as td, timestep, pressure
from tests.fp32_bounds import check_anomaly

pytestmark = pytest.mark.gpu

TOL = {"fp64": 1e-12, "fp32": 1e-5}


def rel_l2(a, b):
    nb = np.linalg.norm(b)
    return np.linalg.norm(a - b) / (nb if nb > 0 else 1.0)


def small_convection(nx=32, ny=32, nz=16, **kw):
    ph = inputs.convection_physics((nx, ny, nz), (2.0 * nx, 2.0 * ny, 1.0 * nz), **kw)
    return ph


def box(n=16, **kw):
    ph = inputs.periodic_box_physics(n)
    for k, v in kw.items():
        setattr(ph, k, v)
    return ph


CASES = {
    "box16_weno5z": lambda: (box(16), lambda ph: inputs.random_state(ph, seed=1)),
    "box32_smooth": lambda: (box(32), lambda ph: inputs.smooth_random_state(ph, seed=2)),
    # convection cases: tracers about the equation of state's reference values
    # (the FP32 storage offsets), velocities of CFL ~ 0.05 at dt = 1 s
    "conv_32x32x16": lambda: (small_convection(), lambda ph: inputs.random_state(
        ph, seed=3, vel=0.1, tracer_means=(ph.t_ref, ph.s_ref))),
    "conv_ragged_64x32x8": lambda: (small_convection(64, 32, 8), lambda ph: inputs.random_state(
        ph, seed=4, vel=0.1, tracer_means=(ph.t_ref, ph.s_ref))),
    "conv_96x16x32_linear": lambda: (small_convection(96, 16, 32, nu=1e-3, kappa=2e-3),
                                    lambda ph: inputs.smooth_random_state(ph, seed=5)),
    "box8_none": lambda: (box(8, advection="none", nu=0.05, kappa=0.01, f=0.3),
                          lambda ph: inputs.random_state(ph, seed=6)),
}


def make_case(name):
    ph, gen = CASES[name]()
    if name.endswith("_linear"):
        ph.advection = "weno5_linear"
    return ph, gen(ph)


def _prep(state, ph, precision):
    """Inputs of the run: the FP32 path starts from the values rounded to FP32."""
    if precision == "fp32":
        return {k: v.astype(np.float32).astype(np.float64) for k, v in state.items()}
    return state


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
def test_set_get_roundtrip(gpu_lib, precision):
    ph, s = make_case("conv_32x32x16")
    m = gpu_lib.Model(ph, precision)
    m.set_states(s)
    for name in m.fields:
        got = m.get_state(name)
        want = s[name].copy()
        if name == "w":
            want[0] = 0.0
            want[-1] = 0.0
        if precision == "fp64":
            assert np.array_equal(got, want), name
        else:
            # FP32 storage (T, S as anomalies about the EOS reference): one
            # rounding of the stored value
            assert rel_l2(got, want) <= 1e-6, name


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("case", list(CASES))
def test_tendency_parity(gpu_lib, case, precision):
    ph, s = make_case(case)
    s = _prep(s, ph, precision)
    m = gpu_lib.Model(ph, precision)
    m.set_states(s)
    m.tendencies()
    st = timestep.make_state(s, ph)
    G = td.tendencies(st, ph)
    for name in m.fields:
        got = m.get_tendency(name)
        err = rel_l2(got, G[name])
        assert err <= TOL[precision], (case, name, err)


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("case", ["box16_weno5z", "conv_32x32x16", "conv_ragged_64x32x8",
                                  "conv_96x16x32_linear"])
def test_pressure_solve_parity(gpu_lib, case, precision):
    ph, _ = make_case(case)
    s = inputs.random_state(ph, seed=21, divergence_free=False)
    s = _prep(s, ph, precision)
    m = gpu_lib.Model(ph, precision)
    m.set_states(s)
    dt_eff = 0.37
    m.pressure_solve(dt_eff)
    w_in = s["w"].copy()
    if ph.z_bounded:
        w_in[0] = w_in[-1] = 0.0
    u, v, w, p = pressure.project(s["u"], s["v"], w_in, dt_eff, ph)
    pg = m.get_pressure()
    assert rel_l2(pg, p) <= 1e-12, rel_l2(pg, p)
    for name, ref in (("u", u), ("v", v), ("w", w)):
        err = rel_l2(m.get_state(name), ref)
        assert err <= TOL[precision], (name, err)
    if precision == "fp64":
        d = m.diagnostics()
        vmax = max(d["max_u"], d["max_v"], d["max_w"])
        assert d["div_scaled_by_dx"] / vmax < 1e-12


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("case,dt,nsteps", [("box16_weno5z", 0.01, 1), ("conv_32x32x16", 1.0, 1),
                                            ("conv_ragged_64x32x8", 1.0, 3),
                                            ("box8_none", 0.02, 2)])
def test_rk3_step_parity(gpu_lib, case, dt, nsteps, precision):
    ph, s = make_case(case)
    s = _prep(s, ph, precision)
    m = gpu_lib.Model(ph, precision)
    m.set_states(s)
    m.rk3_step(dt, nsteps)
    st = timestep.make_state(s, ph)
    for _ in range(nsteps):
        st, _ = timestep.rk3_step(st, dt, ph)
    for name in m.fields:
        ref = fv.interior(st[name], ph, name)
        got = m.get_state(name)
        err = rel_l2(got, ref)
        assert err <= TOL[precision], (case, name, err)
        check_anomaly(got, ref, fv.interior(timestep.make_state(s, ph)[name], ph, name), nsteps,
                      ph, name, precision, case)


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
def test_periodic_box_ten_steps(gpu_lib, precision):
    """Triply periodic 32^3 box: WENO5-Z, nu = kappa = 1e-3, dt = 0.01, 10 RK3 steps."""
    ph = inputs.periodic_box_physics(32)
    s = _prep(inputs.periodic_box_initial(ph, seed=0), ph, precision)
    m = gpu_lib.Model(ph, precision)
    m.set_states(s)
    m.rk3_step(0.01, 10)
    st0 = timestep.make_state(s, ph)
    st = timestep.run(st0, 0.01, 10, ph)
    for name in m.fields:
        ref = fv.interior(st[name], ph, name)
        got = m.get_state(name)
        err = rel_l2(got, ref)
        assert err <= TOL[precision], (name, err)
        check_anomaly(got, ref, fv.interior(st0[name], ph, name), 10, ph, name, precision)


def test_convection_ten_steps_fp64_and_fp32(gpu_lib):
    """Free convection, 64 x 64 x 32 at 2 m x 2 m x 1 m, 10 steps of 1 s:
    FP64 and FP32-mixed against the same FP64 oracle run (per precision, from
    that precision's initial values).  Velocity noise 0.05 m/s and tracer
    noise 0.05 (K, g/kg) on the stratified T and uniform S, so every field,
    S included, changes by percents over the run and its anomaly is held to
    about 1e-5."""
    ph = small_convection(64, 64, 32)
    s = inputs.convection_initial(ph, seed=7, noise=0.05, tracer_noise=0.05)
    for precision in ("fp64", "fp32"):
        s_p = _prep(s, ph, precision)
        st0 = timestep.make_state(s_p, ph)
        st = timestep.run(st0, 1.0, 10, ph)
        m = gpu_lib.Model(ph, precision)
        m.set_states(s_p)
        m.rk3_step(1.0, 10)
        for name in m.fields:
            ref = fv.interior(st[name], ph, name)
            got = m.get_state(name)
            err = rel_l2(got, ref)
            assert err <= TOL[precision], (precision, name, err)
            check_anomaly(got, ref, fv.interior(st0[name], ph, name), 10, ph, name, precision)


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
def test_multi_step_graph_replays_match_direct_launches(gpu_lib, precision):
    """A call of several steps replays a captured step graph (one per buffer
    parity); a single step launches its kernels directly.  Both give the same
    bits after every call: replays of the same graph, a second call that
    reuses the graphs, and a new time step (captured again), with the host
    reading the state between the calls.  The pressure of the last substage,
    which the solve keeps as a spectrum until it is read, is the same too,
    also when the previous call's pressure was read before a replay."""
    ph, s = make_case("conv_32x32x16")
    s = _prep(s, ph, precision)
    direct = gpu_lib.Model(ph, precision)
    direct.set_states(s)
    replay = gpu_lib.Model(ph, precision)
    replay.set_states(s)
    for dt, n in ((1.0, 3), (1.0, 2), (0.5, 3)):
        for _ in range(n):
            direct.rk3_step(dt, 1)
        replay.rk3_step(dt, n)
        for name in direct.fields:
            assert np.array_equal(direct.get_state(name), replay.get_state(name)), (dt, n, name)
        assert np.array_equal(direct.get_pressure(), replay.get_pressure()), (dt, n)


def test_profile_classes_restrict_event_recording(gpu_lib):
    """oc_profile_classes: events around the chosen kernel classes only; the
    default records every class of the step."""
    ph, s = make_case("conv_32x32x16")
    m = gpu_lib.Model(ph, "fp32")
    m.set_states(_prep(s, ph, "fp32"))
    m.profile(True, classes=("tendency",))
    m.rk3_step(1.0, 2)
    m.profile(False)
    p = m.profile_read()
    assert p["tendency"][1] == 6 and p["tendency"][0] > 0
    assert all(n == 0 for k, (_, n) in p.items() if k != "tendency"), p
    m.profile(True)
    m.rk3_step(1.0, 1)
    m.profile(False)
    p = m.profile_read()
    for k in ("tendency", "fft_x_fwd", "fft_y_fwd", "z_solve", "fft_y_inv", "project"):
        assert p[k][1] == 3, (k, p[k])
    assert p["fft_x_inv"][1] == 0   # fused into the projection


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("dtype", ["float32", "float64"])
def test_state_copies_at_element_aligned_addresses(gpu_lib, precision, dtype):
    """Device buffers that start one element into an allocation, on the
    shortest rows and on w's extra level: set and get return the values as
    rounded by the types on the way, and touch nothing beside the buffer."""
    import torch
    ph = inputs.convection_physics((8, 8, 16), (16.0, 16.0, 16.0))
    m = gpu_lib.Model(ph, precision)
    dt = getattr(torch, dtype)
    g = torch.Generator(device="cuda").manual_seed(3)
    for name in m.fields:
        shape = m.shape_of(name)
        n = int(np.prod(shape))
        x = torch.randn(n, generator=g, device="cuda", dtype=torch.float64).to(torch.float32)
        if name == "w":
            x.reshape(shape)[0] = x.reshape(shape)[-1] = 0.0
        buf = torch.full((n + 2,), 7.0, dtype=dt, device="cuda")
        buf[1:-1] = x.to(dt)
        m.set_state(name, buf[1:-1].reshape(shape))
        out = torch.full((n + 2,), 7.0, dtype=dt, device="cuda")
        m.get_state(name, out=out[1:-1].reshape(shape))
        assert float(out[0]) == float(out[-1]) == 7.0
        got = out[1:-1].double()
        # FP32 models keep T and S as anomalies: one rounding of the anomaly
        # (ulp of 35) and one of the value
        tol = 8e-6 if precision == "fp32" and name in ("T", "S") else 0.0
        assert float((got - x.double()).abs().max()) <= tol, name


@pytest.mark.parametrize("n,precision", [((64, 64, 32), "fp32"), ((64, 64, 96), "fp64"),
                                         ((64, 32, 96), "fp64"), ((128, 64, 96), "fp32")])
def test_tendency_parity_by_levels_per_workgroup(gpu_lib, n, precision):
    """Grids whose workgroups walk one, three, two and three levels (the
    latency-bound split), the last chunk shorter where the levels do not
    divide evenly."""
    ph = small_convection(*n)
    s = _prep(inputs.random_state(ph, seed=31, vel=0.1, tracer_means=(ph.t_ref, ph.s_ref)), ph,
              precision)
    m = gpu_lib.Model(ph, precision)
    m.set_states(s)
    m.tendencies()
    G = td.tendencies(timestep.make_state(s, ph), ph)
    for name in m.fields:
        err = rel_l2(m.get_tendency(name), G[name])
        assert err <= TOL[precision], (n, name, err)


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("n,advection", [((8, 8, 8), "weno9z"), ((16, 96, 8), "weno5z"),
                                         ((32, 64, 16), "weno5z"), ((64, 16, 32), "weno7z"),
                                         ((96, 32, 16), "weno5z"), ((128, 8, 32), "weno5z"),
                                         ((256, 16, 8), "weno5z")])
def test_projection_row_blocks(gpu_lib, n, advection, precision):
    """The projection at every transform length, with whole and short row
    blocks, axes shorter than two halos, and the halo images it writes: a
    tendency evaluation reads them."""
    ph = small_convection(*n)
    ph.advection = advection
    s = _prep(inputs.random_state(ph, seed=41, vel=0.1, divergence_free=False,
                                  tracer_means=(ph.t_ref, ph.s_ref)), ph, precision)
    m = gpu_lib.Model(ph, precision)
    m.set_states(s)
    m.pressure_solve(0.37)
    w_in = s["w"].copy()
    w_in[0] = w_in[-1] = 0.0
    u, v, w, p = pressure.project(s["u"], s["v"], w_in, 0.37, ph)
    assert rel_l2(m.get_pressure(), p) <= 1e-12
    for name, ref in (("u", u), ("v", v), ("w", w)):
        err = rel_l2(m.get_state(name), ref)
        assert err <= TOL[precision], (n, name, err)
    m.tendencies()
    G = td.tendencies(timestep.make_state({f: m.get_state(f) for f in m.fields}, ph), ph)
    for name in ("u", "v", "w", "T"):
        err = rel_l2(m.get_tendency(name), G[name])
        assert err <= TOL[precision] * (10 if precision == "fp32" else 1), (n, name, err)


@pytest.mark.parametrize("n,tracers,advection,precision", [
    ((8, 8, 8), ("c",), "weno9z", "fp64"), ((16, 8, 8), ("T", "S", "c", "e"), "weno5z", "fp64"),
    ((32, 8, 16), ("T", "S", "c", "e"), "weno5z", "fp32"), ((96, 16, 8), ("T", "S"), "weno7z", "fp64"),
    ((64, 8, 16), ("T", "S", "c"), "weno5z", "fp32"), ((64, 16, 8), ("c",), "weno5z", "fp32")])
def test_tendency_edge_faces(gpu_lib, n, tracers, advection, precision):
    """The faces at the upper edges of a tile, whose fluxes are dealt over the
    threads field by field: every tile, one to four tracers."""
    ph = small_convection(*n, nu=1e-3, kappa=2e-3)
    ph.advection, ph.tracers, ph.buoyancy = advection, tracers, tracers[0] == "T"
    if not ph.buoyancy:
        ph.top_flux = {}
    s = _prep(inputs.random_state(ph, seed=51, vel=0.1,
                                  tracer_means=(ph.t_ref, ph.s_ref, 1.0, 2.0)[:len(tracers)]),
              ph, precision)
    m = gpu_lib.Model(ph, precision)
    m.set_states(s)
    m.tendencies()
    G = td.tendencies(timestep.make_state(s, ph), ph)
    for name in m.fields:
        err = rel_l2(m.get_tendency(name), G[name])
        assert err <= TOL[precision], (n, name, err)


@pytest.mark.parametrize("precision,eps", [("fp32", 3e-20), ("fp32", 1e-15), ("fp64", 5e-155)])
@pytest.mark.parametrize("moving", [False, True])
def test_weno_regulariser_range(gpu_lib, precision, eps, moving):
    """Stencils that are exactly flat, fully or in part, at regularisers down
    to the smallest whose weights the type can hold (16 eps^2 a normal
    number); at rest every momentum stencil is flat.  (Amplitudes of 0.02:
    next to a flat stencil the square of an indicator over eps has to stay
    in range too.  Tracers without a mean: the divergence that rounding the
    velocities leaves, times a mean of 20, is 4e-5 of the tendency in FP32.)"""
    ph = small_convection(32, 16, 16)
    ph.weno_eps, ph.t_ref, ph.s_ref = eps, 0.0, 0.0
    s = inputs.random_state(ph, seed=61, vel=0.02, tracer_means=(0.0, 0.0), tracer_scale=0.02)
    rng = np.random.default_rng(62)
    for name in ("T", "S"):
        patches = np.repeat(rng.random((ph.nz, ph.ny, ph.nx // 8)) < 0.6, 8, axis=2)
        s[name] = np.where(patches, 0.0, s[name])
    if not moving:
        for name in ("u", "v", "w"):
            s[name] = np.zeros_like(s[name])
    s = _prep(s, ph, precision)
    m = gpu_lib.Model(ph, precision)
    m.set_states(s)
    m.tendencies()
    G = td.tendencies(timestep.make_state(s, ph), ph)
    for name in m.fields:
        err = rel_l2(m.get_tendency(name), G[name])
        assert err <= TOL[precision], (eps, moving, name, err)
