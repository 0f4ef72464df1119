"""GPU parity of the split-explicit barotropic substeps, the baroclinic
correction and the restart against the FP64 oracle (all 2D arithmetic is
FP64: bar 1e-12 relative L2; the corrected 3D velocity is checked at the
precision of the model's state)."""
import numpy as np
import pytest

from paper_2502_14148_amd import inputs
from oracle import free_surface as fso

pytestmark = pytest.mark.gpu


def rel_l2(a, b):
    return np.linalg.norm(a - b) / max(np.linalg.norm(b), 1e-300)


def run_case(gpu_lib, ph, precision, N, M, seed):
    rng = np.random.default_rng(seed + 100)
    b = inputs.barotropic_random_state(ph, seed=seed)
    u = rng.standard_normal((ph.nz, ph.ny, ph.nx)) * 0.1
    v = rng.standard_normal((ph.nz, ph.ny + 1, ph.nx)) * 0.1
    v[:, 0] = 0.0
    v[:, -1] = 0.0
    if precision == "fp32":
        u = u.astype(np.float32).astype(np.float64)
        v = v.astype(np.float32).astype(np.float64)
    w = inputs.averaging_weights(N, M)
    dt = 600.0
    m = gpu_lib.Model(ph, precision)
    for k in ("eta", "U", "V", "GU", "GV"):
        m.set_state(k, b[k])
    m.set_state("u", u)
    m.set_state("v", v)
    m.free_surface_substeps(dt, N, w)
    met = fso.latlon_metrics(ph.nx, ph.ny, ph.lat0, ph.lat_extent, ph.radius, ph.lon_extent)
    e, U, V, eb, ub, vb = fso.substeps(b["eta"][0], b["U"][0], b["V"][0], b["GU"][0], b["GV"][0],
                                       ph.g, ph.depth, dt, N, w, met)
    dz = np.full(ph.nz, ph.depth / ph.nz)
    u_ref = fso.correct_baroclinic(u, dz, ub, ph.depth)
    v_ref = v.copy()
    v_ref[:, 1:-1] = fso.correct_baroclinic(v[:, 1:-1], dz, vb[1:-1], ph.depth)
    got = {k: m.get_state(k)[0] for k in ("eta", "U", "V")}
    for k, ref in (("eta", eb), ("U", ub), ("V", vb)):
        assert rel_l2(got[k], ref) < 1e-12, (k, rel_l2(got[k], ref))
    tol = 1e-12 if precision == "fp64" else 1e-6
    assert rel_l2(m.get_state("u"), u_ref) < tol
    assert rel_l2(m.get_state("v"), v_ref) < tol
    # the corrected baroclinic transport matches the barotropic average
    gu = m.get_state("u")
    assert np.max(np.abs(np.tensordot(dz, gu, axes=(0, 0)) - ub)) < (1e-9 if precision == "fp64" else 1e-2)
    return m


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
def test_substeps_reduced_sector(gpu_lib, precision):
    ph = inputs.sector_physics((144, 56, 10))
    run_case(gpu_lib, ph, precision, N=30, M=59, seed=1)


def test_substeps_ragged_and_single(gpu_lib):
    """Tiles that do not divide the grid, a single substep (M = 1)."""
    ph = inputs.sector_physics((40, 24, 8))
    run_case(gpu_lib, ph, "fp64", N=7, M=1, seed=2)
    run_case(gpu_lib, ph, "fp64", N=5, M=13, seed=3)


def test_substeps_full_sector(gpu_lib):
    """The 1440 x 560 x 50 quarter-degree sector, 30 substeps per 600 s."""
    ph = inputs.sector_physics((1440, 560, 50))
    run_case(gpu_lib, ph, "fp32", N=30, M=59, seed=4)


def test_volume_conserved_on_gpu(gpu_lib):
    ph = inputs.sector_physics((144, 56, 10))
    b = inputs.barotropic_random_state(ph, seed=5)
    m = gpu_lib.Model(ph, "fp64")
    for k in ("eta", "U", "V", "GU", "GV"):
        m.set_state(k, b[k])
    met = fso.latlon_metrics(ph.nx, ph.ny, ph.lat0, ph.lat_extent, ph.radius)
    vol0 = np.sum(met.area[:, None] * b["eta"][0])
    for _ in range(3):
        m.free_surface_substeps(600.0, 30, inputs.averaging_weights(30))
    vol = np.sum(met.area[:, None] * m.get_state("eta")[0])
    assert abs(vol - vol0) < 1e-12 * np.sum(met.area[:, None] * np.abs(b["eta"][0]))


@pytest.mark.parametrize("n,N,M", [((40, 40, 8), 20, 12), ((40, 48, 8), 20, 13),
                                   ((48, 8, 8), 20, 25), ((8, 40, 16), 10, 1),
                                   ((88, 80, 72), 20, 24)])
def test_substeps_tile_edges(gpu_lib, n, N, M):
    """Domains of exactly one 40 x 40 own tile, of a little more, narrower
    than the widened tile (x wraps more than once), and counts of substeps
    around whole launches of 12."""
    run_case(gpu_lib, inputs.sector_physics(n), "fp64", N, M, seed=11)


def test_substeps_without_gravity(gpu_lib):
    """g = 0: the transports move under the forcing alone."""
    ph = inputs.sector_physics((48, 16, 8))
    ph.g = 0.0
    run_case(gpu_lib, ph, "fp64", 10, 19, seed=12)
