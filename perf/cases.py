"""What users of this framework have it do, as cases whose speed is measured.

Every case goes through the public entry points of `paper_2502_14148_amd`:
the nonhydrostatic step (`Model.rk3_step`) with its advection orders,
precisions, vertical grids, closures and boundaries; the hydrostatic step;
ensembles; and the learned closure's network alone and inside the model.  A
pass of a model case advances the model by a few steps and reads the whole
state back into device tensors, as a program does between two outputs.

`exact` states the same computations in 64 bits with plain torch.
"""
import math
from fractions import Fraction

import numpy as np
import torch

from paper_2502_14148_amd import inputs, oc

LENGTHS = (8, 16, 32, 64, 96, 128, 256)     # grid lengths the FFT solver takes
DEV = "cuda:0"


def listed():
    return [
        # the smallest model in use: the triply periodic box of the parity
        # runs, one step per call, where launches and latency count
        _step("box_32_fp64", "periodic", 32, 32, 32, "fp64", steps=1),
        # an ordinary FP64 run on a grid with unequal lengths (96 = 2^5 3)
        _step("convection_96x64x128_fp64", "convection", 96, 64, 128, "fp64", steps=2),
        # the headline workload: 256^3 free convection, FP32 state
        _step("convection_256_fp32", "convection", 256, 256, 256, "fp32", steps=4),
        # the high-order advection of the paper's examples
        _step("convection_128_weno9_fp32", "convection", 128, 128, 128, "fp32", steps=2,
              advection="weno9z"),
        # surface-refined vertical grid with vertically implicit diffusion
        _step("stretched_256x256x128_fp32", "stretched", 256, 256, 128, "fp32", steps=2),
        # free convection with an eddy-viscosity closure
        _step("smagorinsky_256x256x128_fp32", "convection", 256, 256, 128, "fp32", steps=2,
              les="smagorinsky"),
        # flow over a seamount: immersed boundary, iterative pressure solve
        _step("seamount_128_fp32", "seamount", 128, 128, 128, "fp32", steps=1),
        # quarter-degree ocean sector, hydrostatic, split-explicit free surface
        {"name": "sector_1440x560x50_fp32", "kind": "hydrostatic", "nx": 1440, "ny": 560,
         "nz": 50, "precision": "fp32", "steps": 2, "N": 30},
        # a parameter study: uneven members stepped together
        {"name": "ensemble_12_uneven_fp32", "kind": "ensemble", "sizes": "64,96,128",
         "per_size": 4, "precision": "fp32", "steps": 2},
        # inference of the closure network over a 64^3 grid's cells
        {"name": "network_forward_262144", "kind": "forward", "batch": 262144},
        # one training batch of the closure network
        {"name": "network_gradients_4096", "kind": "gradients", "batch": 4096},
        # a coarse model with the learned closure in its tendencies
        {"name": "learned_closure_64_fp32", "kind": "closure", "nx": 64, "ny": 64, "nz": 64,
         "precision": "fp32", "steps": 2},
    ]


def _step(name, grid, nx, ny, nz, precision, steps, advection="weno5z", les="none"):
    return {"name": name, "kind": "step", "grid": grid, "nx": nx, "ny": ny, "nz": nz,
            "precision": precision, "advection": advection, "les": les, "steps": steps}


def draw(rng):
    kind = rng.choice(["step"] * 6 + ["seamount", "hydrostatic", "ensemble", "forward",
                                      "gradients", "closure"])
    prec = rng.choice(["fp32", "fp32", "fp64"])
    if kind == "step":
        while True:
            n = [rng.choice(LENGTHS[1:]), rng.choice(LENGTHS[1:]), rng.choice(LENGTHS)]
            grid = rng.choice(["convection", "convection", "stretched", "periodic"])
            adv = rng.choice(["weno5z"] * 4 + ["weno7z", "weno9z"])
            les = "none"
            if grid == "convection" and adv == "weno5z":
                les = rng.choice(["none", "none", "smagorinsky", "amd"])
            cost = (2 if prec == "fp64" else 1) * {"weno5z": 1, "weno7z": 1.6, "weno9z": 2}[adv]
            if les != "none" or grid == "stretched":
                cost *= 2
            if cost * n[0] * n[1] * n[2] <= 256 ** 3:
                break
        c = _step("", grid, *n, prec, rng.randint(1, 4), adv, les)
        del c["name"]
        return c
    if kind == "seamount":
        n = [rng.choice((32, 64, 96, 128)) for _ in range(3)]
        c = _step("", "seamount", *n, prec, 1)
        del c["name"]
        return c
    if kind == "hydrostatic":
        nx = 8 * round(math.exp(rng.uniform(math.log(5), math.log(180))))
        ny = 8 * round(math.exp(rng.uniform(math.log(3), math.log(70))))
        return {"kind": kind, "nx": nx, "ny": ny, "nz": rng.randint(8, 50), "precision": "fp32",
                "steps": rng.randint(1, 2), "N": rng.choice((10, 20, 30))}
    if kind == "ensemble":
        sizes = sorted(rng.sample((32, 64, 96, 128), rng.randint(1, 3)))
        return {"kind": kind, "sizes": ",".join(str(s) for s in sizes),
                "per_size": rng.randint(1, 4), "precision": "fp32", "steps": rng.randint(1, 2)}
    if kind == "closure":
        return {"kind": kind, "nx": rng.choice((32, 64, 96)), "ny": rng.choice((32, 64)),
                "nz": rng.choice((16, 32, 64)), "precision": "fp32", "steps": rng.randint(1, 2)}
    top = 262144 if kind == "forward" else 16384
    return {"kind": kind,
            "batch": 32 * round(math.exp(rng.uniform(math.log(4), math.log(top // 32))))}


# ---------------------------------------------------------------------------
# Physics and inputs (from the case and the seed alone)
# ---------------------------------------------------------------------------

def _params(case):
    """Parameters of a nonhydrostatic case, as keywords of inputs.Physics."""
    nx, ny, nz = case["nx"], case["ny"], case["nz"]
    grid = case.get("grid", "convection")
    if grid == "periodic":
        length = 2.0 * math.pi
        return dict(nx=nx, ny=ny, nz=nz, lx=length, ly=length, lz=length, z_bounded=False,
                    advection=case["advection"], nu=1e-3, kappa=1e-3, tracers=("c",))
    lz = 1.0 * nz
    p = dict(nx=nx, ny=ny, nz=nz, lx=2.0 * nx, ly=2.0 * ny, lz=lz, z_bounded=True, z0=-lz,
             advection=case.get("advection", "weno5z"), f=1e-4, g=9.81, alpha=2e-4, beta=8e-4,
             t_ref=20.0, s_ref=35.0, nu=1e-5, kappa=1e-5, tracers=("T", "S"), buoyancy=True,
             top_flux={"T": case.get("flux", 1e-8) / (9.81 * 2e-4)},
             les=case.get("les", "none"), closure=case["kind"] == "closure")
    if grid == "stretched":
        zf = -lz + lz * np.tanh(1.5 * np.arange(nz + 1) / nz) / np.tanh(1.5)
        zf[0], zf[-1] = -lz, 0.0
        p.update(z_faces=tuple(float(z) for z in zf), implicit_z=True)
    if grid == "seamount":
        x = (np.arange(nx) + 0.5) / nx - 0.5
        y = (np.arange(ny) + 0.5) / ny - 0.5
        h = 0.4 * np.exp(-(x[None, :] ** 2 + y[:, None] ** 2) / (2 * 0.15 ** 2))
        z = (np.arange(nz) + 0.5) / nz
        p.update(solid=z[:, None, None] < h[None], cg_tol=1e-10 if case["precision"] == "fp32"
                 else 1e-13)
    return p


def _dt(case):
    return 0.01 if case.get("grid") == "periodic" else 1.0


def _generator(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(int(seed) * 2654435761 % (1 << 62) + 17)
    return g


def _dtype(case):
    return torch.float64 if case["precision"] == "fp64" else torch.float32


def _fields(case, p, seed):
    """Initial state: a divergence-free random velocity (curl of a random edge
    potential), a stratified T (or blobs of c) with noise, S with noise."""
    g = _generator(seed)
    nx, ny, nz = p["nx"], p["ny"], p["nz"]
    bounded = p["z_bounded"]
    nw = nz + 1 if bounded else nz
    kw = dict(generator=g, device=DEV, dtype=torch.float64)
    dx, dy = p["lx"] / nx, p["ly"] / ny
    zf = torch.tensor(p["z_faces"], device=DEV, dtype=torch.float64) if p.get("z_faces") else \
        p.get("z0", 0.0) + torch.arange(nz + 1, device=DEV, dtype=torch.float64) * (p["lz"] / nz)
    dz = (zf[1:] - zf[:-1])[:, None, None]
    ax, ay = torch.randn((nw, ny, nx), **kw), torch.randn((nw, ny, nx), **kw)
    az = torch.randn((nz, ny, nx), **kw)
    if not bounded:      # a smooth flow: a few large scales
        for a in (ax, ay, az):
            s = torch.fft.fftn(a)
            k = [torch.fft.fftfreq(n, d=1.0 / n, device=DEV, dtype=torch.float64)
                 for n in a.shape]
            k2 = k[0][:, None, None] ** 2 + k[1][None, :, None] ** 2 + k[2][None, None, :] ** 2
            s *= ((k2 > 0) & (k2 <= 64)) / (1.0 + k2) ** 1.8
            a.copy_(torch.fft.ifftn(s).real)
    else:
        ax[0] = ax[-1] = 0.0
        ay[0] = ay[-1] = 0.0

    def up(a, d):
        return torch.roll(a, -1, d) - a

    def dzf(a):
        return (a[1:] - a[:-1]) / dz if bounded else up(a, 0) / dz
    u = up(az, 1) / dy - dzf(ay)
    v = dzf(ax) - up(az, 2) / dx
    w = up(ay, 2) / dx - up(ax, 1) / dy
    rms = torch.sqrt((u.square().mean() + v.square().mean() + w.square().mean()) / 3)
    scale = (1e-3 if bounded else 1.0) / rms
    out = {"u": u * scale, "v": v * scale, "w": w * scale}
    if bounded:
        out["w"][0] = 0.0
        out["w"][-1] = 0.0
        zc = 0.5 * (zf[1:] + zf[:-1])
        T = (20.0 + 1e-5 / (9.81 * 2e-4) * zc)[:, None, None]
        out["T"] = T + 1e-3 * torch.randn((nz, ny, nx), **kw)
        out["S"] = 35.0 + 1e-3 * torch.randn((nz, ny, nx), **kw)
    else:
        c = torch.zeros((nz, ny, nx), device=DEV, dtype=torch.float64)
        at = torch.rand((8, 3), **kw)
        for b in range(8):
            r2 = 0.0
            for axis, n in enumerate((nz, ny, nx)):
                x = (torch.arange(n, device=DEV, dtype=torch.float64) + 0.5) / n - at[b, axis]
                x = (x - torch.round(x)) * p["lx"]
                shape = [1, 1, 1]
                shape[axis] = n
                r2 = r2 + x.reshape(shape) ** 2
            c += torch.exp(-r2 / (2 * 0.3 ** 2))
        out["c"] = c
    return {k: a.to(_dtype(case)).contiguous() for k, a in out.items()}


def _sector_fields(case, seed):
    """Sector state: linear T profile with noise, S = 35 with noise, a smooth
    flow with its depth integrals, zonal wind bands."""
    g = _generator(seed)
    kw = dict(generator=g, device=DEV, dtype=torch.float64)
    nx, ny, nz = case["nx"], case["ny"], case["nz"]
    depth = 3000.0
    z = -depth + (torch.arange(nz, device=DEV, dtype=torch.float64) + 0.5) * (depth / nz)
    T = (2.0 + 18.0 * (1.0 + z / depth))[:, None, None] + 0.1 * torch.randn((nz, ny, nx), **kw)
    S = 35.0 + 0.01 * torch.randn((nz, ny, nx), **kw)
    lam = 2 * math.pi * torch.arange(nx, device=DEV, dtype=torch.float64) / nx
    yc = (torch.arange(ny, device=DEV, dtype=torch.float64) + 0.5) / ny
    yf = torch.arange(ny + 1, device=DEV, dtype=torch.float64) / ny
    u = torch.zeros((nz, ny, nx), device=DEV, dtype=torch.float64)
    v = torch.zeros((nz, ny + 1, nx), device=DEV, dtype=torch.float64)
    c = torch.rand((4, 4), **kw)
    for q in range(4):
        zs = torch.cos(q * math.pi * (z + depth) / depth + 6 * c[q, 0])[:, None, None]
        wave = torch.cos((1 + q % 3) * lam + 6 * c[q, 1])[None, None, :]
        u += 0.03 * zs * wave * torch.cos((1 + q % 2) * math.pi * yc + 6 * c[q, 2])[None, :, None]
        v += 0.03 * zs * wave * torch.sin((1 + q % 3) * math.pi * yf)[None, :, None]
    v[:, 0] = 0.0
    v[:, ny] = 0.0
    a = 0.05 / 1026.0 * torch.randn(6, **kw)
    tau = sum(a[m] * torch.sin((m + 1) * math.pi * yc) for m in range(6))
    out = {"u": u, "v": v, "T": T, "S": S}
    out = {k: x.to(_dtype(case)).contiguous() for k, x in out.items()}
    dz = depth / nz
    out["eta"] = torch.zeros((1, ny, nx), device=DEV, dtype=torch.float64)
    out["U"] = dz * out["u"].double().sum(0, keepdim=True)
    out["V"] = dz * out["v"].double().sum(0, keepdim=True)
    out["tau_x"] = (tau[:, None] * torch.ones((1, nx), device=DEV, dtype=torch.float64))[None]
    out["tau_y"] = torch.zeros((1, ny + 1, nx), device=DEV, dtype=torch.float64)
    return {k: x.contiguous() for k, x in out.items()}


def _network(seed):
    """Weights N(0, 1/fan_in), small biases; FP32 values on the host."""
    r = np.random.default_rng(int(seed) + 5)
    p = {}
    for k, shp in (("W1", (256, 500)), ("b1", (256,)), ("W2", (256, 256)), ("b2", (256,)),
                   ("W3", (4, 256)), ("b3", (4,))):
        s = 1.0 / math.sqrt(shp[1]) if len(shp) == 2 else 0.05
        p[k] = (s * r.standard_normal(shp)).astype(np.float32)
    return p


#: means and standard deviations of (u, v, w, b), then of the four fluxes
STATS = np.array([0.0, 0.0, 0.0, -3e-4] + [1e-3, 1e-3, 1e-3, 2e-4]
                 + [0.0] * 4 + [1e-7, 1e-7, 1e-7, 1e-9])


def _batch(case, seed):
    g = _generator(seed)
    x = torch.randn((case["batch"], 500), generator=g, device=DEV)
    t = torch.randn((case["batch"], 4), generator=g, device=DEV)
    return x, t


def _members(case, seed):
    """(case, seed) of each member of an ensemble: free convection at N^3
    with its own surface buoyancy flux."""
    r = np.random.default_rng(int(seed) + 3)
    out = []
    for n in (int(s) for s in case["sizes"].split(",")):
        for _ in range(case["per_size"]):
            out.append((dict(kind="step", grid="convection", nx=n, ny=n, nz=n,
                             precision=case["precision"], advection="weno5z", les="none",
                             flux=float(r.uniform(0.5e-8, 2e-8))),
                        int(r.integers(0, 1 << 30))))
    return out


# ---------------------------------------------------------------------------
# prepare and run
# ---------------------------------------------------------------------------

def _model(case, seed):
    p = _params(case)
    m = oc.Model(inputs.Physics(**p), case["precision"])
    s = _fields(case, p, seed)
    m.set_states(s)
    return m, {k: torch.empty_like(a) for k, a in s.items()}


def _weights(N):
    return inputs.averaging_weights(N)


def prepare(case, seed):
    kind = case["kind"]
    if kind == "step":
        m, out = _model(case, seed)
        return {"kind": kind, "m": m, "out": out, "dt": _dt(case), "steps": case["steps"]}
    if kind == "closure":
        m, out = _model(case, seed)
        net = oc.Mlp(case["nx"] * case["ny"] * case["nz"])
        net.set_params(_network(seed))
        m.set_closure(net, STATS)
        return {"kind": "step", "m": m, "out": out, "dt": _dt(case), "steps": case["steps"]}
    if kind == "hydrostatic":
        ph = inputs.HydrostaticPhysics(nx=case["nx"], ny=case["ny"], nz=case["nz"])
        m = oc.Model(ph, case["precision"])
        s = _sector_fields(case, seed)
        m.set_states(s)
        for k in ("eta", "U", "V", "tau_x", "tau_y"):
            m.set_state(k, s[k])
        out = {k: torch.empty_like(s[k]) for k in ("u", "v", "T", "S")}
        return {"kind": kind, "m": m, "out": out, "N": case["N"], "w": _weights(case["N"]),
                "steps": case["steps"]}
    if kind == "ensemble":
        ms = [_model(c, s) for c, s in _members(case, seed)]
        return {"kind": kind, "e": oc.Ensemble([m for m, _ in ms], graph=True), "ms": ms,
                "steps": case["steps"]}
    net = oc.Mlp(case["batch"])
    net.set_params(_network(seed))
    x, t = _batch(case, seed)
    return {"kind": kind, "net": net, "x": x, "t": t}


def run(state):
    kind = state["kind"]
    if kind == "step":
        state["m"].rk3_step(state["dt"], state["steps"])
        return _read(state["m"], state["out"])
    if kind == "hydrostatic":
        state["m"].hydrostatic_step(600.0, state["N"], state["w"], state["steps"])
        return _read(state["m"], state["out"])
    if kind == "ensemble":
        state["e"].step(1.0, state["steps"])
        return [_read(m, out) for m, out in state["ms"]]
    if kind == "forward":
        return state["net"].forward(state["x"])
    g, loss = state["net"].gradients(state["x"], state["t"])
    return {"grad": g, "loss": loss}


def _read(m, out):
    for k, a in out.items():
        m.get_state(k, out=a)
    return out


def work(case):
    """Bytes: per substage the state in and out of the tendencies and the
    velocities in and out of the projection (the pressure solve between them
    is global), then the state read out.  Flops: the advection's."""
    kind = case["kind"]
    if kind in ("forward", "gradients"):
        b = case["batch"]
        mul = 2.0 * b * (500 * 256 + 256 * 256 + 256 * 4)
        if kind == "forward":
            return {"bytes": b * 504 * 4.0, "flops": mul}
        return {"bytes": b * 504 * 4.0 + 2 * 195076 * 4.0, "flops": 3 * mul}
    if kind == "ensemble":
        w = [work(dict(c, steps=case["steps"])) for c, _ in _members(case, 0)]
        return {k: sum(x[k] for x in w) for k in ("bytes", "flops")}
    n = float(case["nx"] * case["ny"] * case["nz"])
    esz = 8 if case["precision"] == "fp64" else 4
    if kind == "hydrostatic":
        return {"bytes": n * esz * (case["steps"] * 8 + 8), "flops": n * 914.0 * case["steps"]}
    nf = 4 if case.get("grid") == "periodic" else 5
    flops = {"weno5z": 1373.0, "weno7z": 2375.0, "weno9z": 3767.0}[
        case.get("advection", "weno5z")]
    if kind == "closure":
        flops += 2.0 * (500 * 256 + 256 * 256 + 256 * 4)
    return {"bytes": n * esz * (3 * case["steps"] * (2 * nf + 6) + 2 * nf),
            "flops": n * 3 * case["steps"] * flops}


# ---------------------------------------------------------------------------
# The same in 64 bits, with plain torch
# ---------------------------------------------------------------------------

def exact(case, seed):
    kind = case["kind"]
    if kind == "forward":
        x, _ = _batch(case, seed)
        p = {k: torch.from_numpy(v).to(DEV).double() for k, v in _network(seed).items()}
        return torch.cat([_mlp(p, c.double()) for c in x.split(65536)])
    if kind == "gradients":
        x, t = _batch(case, seed)
        p = {k: torch.from_numpy(v).to(DEV).double().requires_grad_(True)
             for k, v in _network(seed).items()}
        loss = (_mlp(p, x.double()) - t.double()).square().mean()
        g = torch.autograd.grad(loss, list(p.values()))
        return {"grad": torch.cat([a.reshape(-1) for a in g]), "loss": float(loss)}
    if kind == "hydrostatic":
        return _exact_sector(case, seed)
    if kind == "ensemble":
        return [_exact_step(dict(c, steps=case["steps"]), s) for c, s in _members(case, seed)]
    return _exact_step(case, seed)


def _mlp(p, x):
    h = torch.nn.functional.gelu(x @ p["W1"].T + p["b1"])
    h = torch.nn.functional.gelu(h @ p["W2"].T + p["b2"])
    return h @ p["W3"].T + p["b3"]


class _Weno:
    """WENO-Z of order 2r - 1 from its construction: candidate polynomials
    over r cells, ideal weights, Jiang-Shu indicators.  Cell m covers
    [m, m + 1], the interface is at 0."""

    TAU = {3: (1, 0, -1), 4: (1, 3, -3, -1), 5: (1, 2, -6, 2, 1)}

    def __init__(self, r):
        self.r = r

        def inverse(cells):
            n = len(cells)
            a = [[Fraction((m + 1) ** (q + 1) - m ** (q + 1), q + 1) for q in range(n)]
                 for m in cells]
            b = [row + [Fraction(int(i == j)) for j in range(n)] for i, row in enumerate(a)]
            for c in range(n):
                q = next(i for i in range(c, n) if b[i][c] != 0)
                b[c], b[q] = b[q], b[c]
                b[c] = [x / b[c][c] for x in b[c]]
                for i in range(n):
                    if i != c and b[i][c] != 0:
                        b[i] = [x - b[i][c] * y for x, y in zip(b[i], b[c])]
            return [row[n:] for row in b]

        def deriv(q, l):      # l-th derivative of x^q: (factor, power)
            f = 1
            for s in range(l):
                f *= q - s
            return f, q - l
        s_mat = [[Fraction(0)] * r for _ in range(r)]
        for q in range(r):
            for t in range(r):
                for l in range(1, r):
                    (fa, pa), (fb, pb) = deriv(q, l), deriv(t, l)
                    if fa and fb:
                        n = pa + pb + 1
                        s_mat[q][t] += Fraction(fa * fb * (0 - (-1) ** n), n)
        self.cand, self.chol = [], []
        for s in range(r):
            cells = list(range(-r + s, s))
            inv = inverse(cells)
            self.cand.append([float(x) for x in inv[0]])
            q = np.array([[float(sum(inv[a][i] * s_mat[a][b] * inv[b][j] for a in range(r)
                                     for b in range(r))) for j in range(r)] for i in range(r)])
            keep = [i for i, m in enumerate(cells) if m != -1]    # deviations from cell -1
            self.chol.append((keep, np.linalg.cholesky(q[np.ix_(keep, keep)])))
        wide = [float(x) for x in inverse(list(range(-r, r - 1)))[0]]
        a = np.zeros((2 * r - 1, r))
        for s in range(r):
            for i in range(r):
                a[s + i, s] = self.cand[s][i]
        self.ideal = np.linalg.lstsq(a, np.array(wide), rcond=None)[0]

    def __call__(self, vals, vel, eps=1e-15):
        """vals: the 2r values around the face, offsets -r .. r-1."""
        r, pos = self.r, vel > 0
        q = [torch.where(pos, vals[m], vals[2 * r - 1 - m]) for m in range(2 * r - 1)]
        c = q[r - 1]
        d = [x - c for x in q]
        beta = []
        for s in range(r):
            keep, l = self.chol[s]
            b = 0.0
            for j in range(r - 1):
                b = b + sum(float(l[i, j]) * d[s + keep[i]] for i in range(j, r - 1)) ** 2
            beta.append(b)
        tau = sum(t * b for t, b in zip(self.TAU[r], beta) if t).abs()
        num, den = 0.0, 0.0
        for s in range(r):
            a = float(self.ideal[s]) * (1.0 + (tau / (beta[s] + eps)) ** 2)
            num = num + a * sum(float(x) * d[s + i] for i, x in enumerate(self.cand[s]))
            den = den + a
        return c + num / den


_CENTRED = {2: (0.5, 0.5), 4: (-1 / 12, 7 / 12, 7 / 12, -1 / 12),
            6: (1 / 60, -8 / 60, 37 / 60, 37 / 60, -8 / 60, 1 / 60),
            8: (-3 / 840, 29 / 840, -139 / 840, 533 / 840, 533 / 840, -139 / 840, 29 / 840,
                -3 / 840)}
_H = 5


def _index(n, bounded, face):
    """Source index and sign of the padded positions -H .. n + H - 1 (+1)."""
    i = torch.arange(-_H, n + _H, device=DEV)
    if not bounded:
        return i % n, None
    if not face:
        return torch.where(i < 0, -1 - i, torch.where(i >= n, 2 * n - 1 - i, i)), None
    s = torch.where((i < 0) | (i > n), -1.0, 1.0).double()
    s[(i == 0) | (i == n)] = 0.0
    return torch.where(i < 0, -i, torch.where(i > n, 2 * n - i, i)), s


def _pad(a, zb, face=False):
    """Halo of width H: periodic x, y; z periodic or mirrored (oddly for w)."""
    nz = a.shape[0] - 1 if (zb and face) else a.shape[0]
    k, s = _index(nz, zb, face)
    a = a.index_select(0, k)
    if s is not None:
        a = a * s[:, None, None]
    for d in (1, 2):
        a = a.index_select(d, _index(a.shape[d], False, False)[0])
    return a


class _Box:
    """The nonhydrostatic discretisation on interior arrays (k, j, i)."""

    def __init__(self, p):
        self.p = p
        self.nx, self.ny, self.nz, self.zb = p["nx"], p["ny"], p["nz"], p["z_bounded"]
        self.dx, self.dy = p["lx"] / self.nx, p["ly"] / self.ny
        r = {"weno5z": 3, "weno7z": 4, "weno9z": 5}[p["advection"]]
        self.r, self.weno, self.cen = r, _Weno(r), _CENTRED[2 * r - 2]
        kw = dict(device=DEV, dtype=torch.float64)
        nz = self.nz
        if p.get("z_faces"):
            zf = torch.tensor(p["z_faces"], **kw)
            dzc = zf[1:] - zf[:-1]
            dzf = torch.cat([dzc[:1], 0.5 * (dzc[1:] + dzc[:-1]), dzc[-1:]])
        else:
            dzc = torch.full((nz,), p["lz"] / nz, **kw)
            dzf = torch.full((nz + 1,), p["lz"] / nz, **kw)
        self.dzc, self.dzf = dzc[:, None, None], dzf[:, None, None]
        self.solid = None
        if p.get("solid") is not None:
            c = 1.0 - torch.from_numpy(np.ascontiguousarray(p["solid"])).to(DEV).double()
            self.solid = c
            oz = torch.zeros((nz + 1, self.ny, self.nx), **kw)
            oz[1:nz] = c[1:] * c[:-1]
            self.open = (c * torch.roll(c, 1, 2), c * torch.roll(c, 1, 1), oz)
        # pressure operator: Fourier in x, y; along z Fourier or the
        # eigenvectors of the symmetrised vertical operator
        sx = torch.sin(math.pi * torch.arange(self.nx, **kw) / self.nx) * 2 / self.dx
        sy = torch.sin(math.pi * torch.arange(self.ny, **kw) / self.ny) * 2 / self.dy
        lxy = -(sy[:, None] ** 2 + sx[None, :] ** 2)
        if self.zb:
            off = 1.0 / dzf[1:nz]
            a = torch.diag(off, 1) + torch.diag(off, -1)
            a = a - torch.diag(a.sum(1))
            h = 1.0 / torch.sqrt(dzc)
            ev, vec = torch.linalg.eigh((a * h[:, None] * h[None, :]).cpu())
            lz, self.vec, self.h = ev.to(DEV), vec.to(DEV), h
            lz[-1] = 0.0                     # the constant mode
            zero = nz - 1
        else:
            lz = -(torch.sin(math.pi * torch.arange(nz, **kw) / nz) * 2 * nz / p["lz"]) ** 2
            zero = 0
        lam = lz[:, None, None] + lxy[None]
        lam[zero, 0, 0] = 1.0
        self.rlam = 1.0 / lam
        self.rlam[zero, 0, 0] = 0.0

    def mm(self, m, a):
        return (m @ a.reshape(a.shape[0], -1)).reshape(a.shape)

    def poisson(self, rhs):
        if not self.zb:
            return torch.fft.ifftn(torch.fft.fftn(rhs) * self.rlam).real
        a = self.mm(self.vec.T.contiguous(), rhs / self.h[:, None, None])
        a = torch.fft.ifft2(torch.fft.fft2(a) * self.rlam).real
        return self.mm(self.vec, a) * self.h[:, None, None]

    # block of a padded array: interior start offset and extra extent
    def blk(self, a, d=(0, 0, 0), e=(0, 0, 0)):
        n = (self.nz, self.ny, self.nx)
        return a[tuple(slice(_H + d[q], _H + d[q] + n[q] + e[q]) for q in range(3))]

    def shifts(self, a, axis, offs, e):
        return [self.blk(a, tuple(o if q == axis else 0 for q in range(3)), e) for o in offs]

    def rec(self, a, axis, vel, e):
        return self.weno(self.shifts(a, axis, range(-self.r, self.r), e), vel)

    def mid(self, a, axis, e):
        n = len(self.cen) // 2
        v = self.shifts(a, axis, range(-n, n), e)
        return sum(c * x for c, x in zip(self.cen, v))

    def dif(self, a, axis, e):
        lo, hi = self.shifts(a, axis, (-1, 0), e)
        return hi - lo

    def flux_div(self, fx, fy, fz, hz):
        return ((fx[:, :, 1:] - fx[:, :, :-1]) / self.dx + (fy[:, 1:] - fy[:, :-1]) / self.dy
                + (fz[1:] - fz[:-1]) / hz)

    def tendencies(self, s):
        p, zb, nz = self.p, self.zb, self.nz
        E = ((0, 0, 1), (0, 1, 0), (1, 0, 0))        # one more face along x, y, z
        P = {k: _pad(a, zb, k == "w") for k, a in s.items()}
        u, v, w = P["u"], P["v"], P["w"]
        nu, ka = p["nu"], p["kappa"]
        nuz, kaz = (0.0, 0.0) if p.get("implicit_z") else (nu, ka)
        op = (1.0, 1.0, 1.0)
        if self.solid is not None:
            ox, oy, oz = self.open
            op = (torch.cat([ox, ox[:, :, :1]], 2), torch.cat([oy, oy[:, :1]], 1), oz)
        G = {}
        for q, n in enumerate(p["tracers"]):
            c = P[n]
            vx, vy, vz = self.blk(u, e=E[0]), self.blk(v, e=E[1]), self.blk(w, e=E[2])
            fx = vx * self.rec(c, 2, vx, E[0]) - op[0] * ka * self.dif(c, 2, E[0]) / self.dx
            fy = vy * self.rec(c, 1, vy, E[1]) - op[1] * ka * self.dif(c, 1, E[1]) / self.dy
            fz = vz * self.rec(c, 0, vz, E[2]) - op[2] * kaz * self.dif(c, 0, E[2]) / self.dzf
            if zb:
                fz[0] = 0.0
                fz[nz] = p.get("top_flux", {}).get(n, 0.0) * \
                    (self.solid[nz - 1] if self.solid is not None else 1.0)
            G[n] = -self.flux_div(fx, fy, fz, self.dzc)
        # u
        a = self.mid(u, 2, E[0])
        fx = a * self.rec(u, 2, a, E[0]) - nu * self.dif(u, 2, E[0]) / self.dx
        a = self.mid(v, 2, E[1])
        fy = a * self.rec(u, 1, a, E[1]) - nu * self.dif(u, 1, E[1]) / self.dy
        a = self.mid(w, 2, E[2])
        fz = a * self.rec(u, 0, a, E[2]) - nuz * self.dif(u, 0, E[2]) / self.dzf
        if zb:
            fz[0] = fz[nz] = 0.0
        G["u"] = -self.flux_div(fx, fy, fz, self.dzc)
        # v
        a = self.mid(u, 1, E[0])
        fx = a * self.rec(v, 2, a, E[0]) - nu * self.dif(v, 2, E[0]) / self.dx
        a = self.mid(v, 1, E[1])
        fy = a * self.rec(v, 1, a, E[1]) - nu * self.dif(v, 1, E[1]) / self.dy
        a = self.mid(w, 1, E[2])
        fz = a * self.rec(v, 0, a, E[2]) - nuz * self.dif(v, 0, E[2]) / self.dzf
        if zb:
            fz[0] = fz[nz] = 0.0
        G["v"] = -self.flux_div(fx, fy, fz, self.dzc)
        # w
        a = self.mid(u, 0, E[0])
        fx = a * self.rec(w, 2, a, E[0]) - nu * self.dif(w, 2, E[0]) / self.dx
        a = self.mid(v, 0, E[1])
        fy = a * self.rec(w, 1, a, E[1]) - nu * self.dif(w, 1, E[1]) / self.dy
        a = self.mid(w, 0, E[2])
        below = self.dzc[:1] if zb else self.dzc[-1:]
        fz = a * self.rec(w, 0, a, E[2]) - nuz * self.dif(w, 0, E[2]) / \
            torch.cat([below, self.dzc])
        gw = -self.flux_div(fx, fy, fz, self.dzf[:nz])
        if p.get("buoyancy"):
            b = p["g"] * (p["alpha"] * (P["T"] - p["t_ref"]) - p["beta"] * (P["S"] - p["s_ref"]))
            gw = gw + 0.5 * (self.blk(b, (-1, 0, 0)) + self.blk(b))
        f = p.get("f", 0.0)
        if f:
            G["u"] = G["u"] + f * 0.25 * sum(self.blk(v, (0, j, i)) for j in (0, 1)
                                             for i in (-1, 0))
            G["v"] = G["v"] - f * 0.25 * sum(self.blk(u, (0, j, i)) for j in (-1, 0)
                                             for i in (0, 1))
        if zb:
            gw = torch.cat([gw, torch.zeros_like(gw[:1])])
            gw[0] = 0.0
        G["w"] = gw
        if p.get("les", "none") != "none":
            for k, a in self.les(P).items():
                G[k] = G[k] + a
        if self.solid is not None:
            for k, o in zip("uvw", self.open):
                G[k] = G[k] * o
        return G


    # ---- eddy-viscosity closures
    def les(self, P):
        p, nz, zb = self.p, self.nz, self.zb
        u, v, w = P["u"], P["v"], P["w"]
        dx, dy = self.dx, self.dy

        def d(a, axis, h, e):
            return self.dif(a, axis, e) / h
        ux = (self.blk(u, (0, 0, 1)) - self.blk(u)) / dx
        vy = (self.blk(v, (0, 1, 0)) - self.blk(v)) / dy
        wz = (self.blk(w, (1, 0, 0)) - self.blk(w)) / self.dzc
        xy, xz, yz = (0, 1, 1), (1, 0, 1), (1, 1, 0)
        uy, vx = d(u, 1, dy, xy), d(v, 2, dx, xy)
        uz, wx = d(u, 0, self.dzf, xz), d(w, 2, dx, xz)
        vz, wy = d(v, 0, self.dzf, yz), d(w, 1, dy, yz)
        for a in (uz, wx, vz, wy):
            if zb:
                a[0] = a[nz] = 0.0

        def axy(a):
            return 0.25 * (a[:, :-1, :-1] + a[:, 1:, :-1] + a[:, :-1, 1:] + a[:, 1:, 1:])

        def axz(a):
            return 0.25 * (a[:-1, :, :-1] + a[1:, :, :-1] + a[:-1, :, 1:] + a[1:, :, 1:])

        def ayz(a):
            return 0.25 * (a[:-1, :-1] + a[1:, :-1] + a[:-1, 1:] + a[1:, 1:])

        def gradz(c):
            g = d(c, 0, self.dzf, (1, 0, 0))
            if zb:
                g[0] = g[nz] = 0.0
            return 0.5 * (g[1:] + g[:-1])
        if p["les"] == "smagorinsky":
            s2 = 2 * (ux ** 2 + vy ** 2 + wz ** 2) + \
                (axy((uy + vx) ** 2) + axz((uz + wx) ** 2) + ayz((vz + wy) ** 2))
            b = p["g"] * (p["alpha"] * (P["T"] - p["t_ref"]) - p["beta"] * (P["S"] - p["s_ref"]))
            n2 = gradz(b)
            safe = torch.where(s2 > 0, s2, torch.ones_like(s2))
            fac = torch.where(s2 > 0, (1.0 - n2 / safe).clamp(min=0.0), torch.zeros_like(s2))
            nue = 0.16 ** 2 * (dx * dy * self.dzc) ** (2.0 / 3.0) * torch.sqrt(s2) * torch.sqrt(fac)
            kap = {n: nue for n in p["tracers"]}
        else:
            g = [[ux, axy(uy), axz(uz)], [axy(vx), vy, ayz(vz)], [axz(wx), ayz(wy), wz]]
            D2 = [dx * dx, dy * dy, self.dzc ** 2]
            num = sum(D2[k] * g[i][k] * g[j][k] * 0.5 * (g[i][j] + g[j][i])
                      for k in range(3) for i in range(3) for j in range(3))
            den = sum(g[i][k] ** 2 for i in range(3) for k in range(3))
            nue = torch.where(den > 0, -num / 12.0 / torch.where(den > 0, den, 1.0),
                              0.0).clamp(min=0.0)
            kap = {}
            for n in p["tracers"]:
                fx, fy = d(P[n], 2, dx, (0, 0, 1)), d(P[n], 1, dy, (0, 1, 0))
                gc = [0.5 * (fx[:, :, 1:] + fx[:, :, :-1]), 0.5 * (fy[:, 1:] + fy[:, :-1]),
                      gradz(P[n])]
                num = sum(D2[k] * g[i][k] * gc[k] * gc[i] for k in range(3) for i in range(3))
                den = gc[0] ** 2 + gc[1] ** 2 + gc[2] ** 2
                kap[n] = torch.where(den > 0, -num / 12.0 / torch.where(den > 0, den, 1.0),
                                     0.0).clamp(min=0.0)
        N = _pad(nue, zb)

        def edge(a, b, e):      # mean of the four centres around an edge
            zero = [0, 0, 0]
            pts = []
            for i in (0, -1):
                for j in (0, -1):
                    o = list(zero)
                    o[a], o[b] = i, j
                    pts.append(self.blk(N, tuple(o), e))
            return 0.25 * sum(pts)
        txx, tyy, tzz = 2 * nue * ux, 2 * nue * vy, 2 * nue * wz
        txy = edge(1, 2, xy) * (uy + vx)
        txz = edge(0, 2, xz) * (uz + wx)
        tyz = edge(0, 1, yz) * (vz + wy)
        out = {}
        out["u"] = ((txx - torch.roll(txx, 1, 2)) / dx + (txy[:, 1:, :-1] - txy[:, :-1, :-1]) / dy
                    + (txz[1:, :, :-1] - txz[:-1, :, :-1]) / self.dzc)
        out["v"] = ((txy[:, :-1, 1:] - txy[:, :-1, :-1]) / dx + (tyy - torch.roll(tyy, 1, 1)) / dy
                    + (tyz[1:, :-1] - tyz[:-1, :-1]) / self.dzc)
        low = torch.cat([tzz[:1] if zb else tzz[-1:], tzz[:-1]])
        gw = ((txz[:nz, :, 1:] - txz[:nz, :, :-1]) / dx + (tyz[:nz, 1:] - tyz[:nz, :-1]) / dy
              + (tzz - low) / self.dzf[:nz])
        if zb:
            gw = torch.cat([gw, torch.zeros_like(gw[:1])])
            gw[0] = 0.0
        out["w"] = gw
        for n in p["tracers"]:
            K, c = _pad(kap[n], zb), P[n]

            def face(axis, e):
                a, b = self.shifts(K, axis, (-1, 0), e)
                return 0.5 * (a + b)
            fx = face(2, (0, 0, 1)) * d(c, 2, dx, (0, 0, 1))
            fy = face(1, (0, 1, 0)) * d(c, 1, dy, (0, 1, 0))
            fz = face(0, (1, 0, 0)) * d(c, 0, self.dzf, (1, 0, 0))
            if zb:
                fz[0] = fz[nz] = 0.0
            out[n] = self.flux_div(fx, fy, fz, self.dzc)
        return out

    # ---- vertically implicit diffusion: (1 - dt d/dz K d/dz) x = x~
    def implicit(self, s, dt):
        p, nz = self.p, self.nz
        dzc, dzf = self.dzc.reshape(-1), self.dzf.reshape(-1)
        eye = torch.eye(nz, device=DEV, dtype=torch.float64)

        def centred(K):
            f = K / dzf[1:nz]
            a = torch.diag(f, 1) + torch.diag(f, -1)
            return torch.linalg.inv(eye - dt * (a - torch.diag(a.sum(1))) / dzc[:, None])
        f = p["nu"] / dzc
        a = torch.diag(f[1:-1], 1) + torch.diag(f[1:-1], -1) - torch.diag(f[1:] + f[:-1])
        faces = torch.linalg.inv(eye[1:, 1:] - dt * a / dzf[1:nz, None])
        m = {"u": centred(p["nu"]), "v": centred(p["nu"])}
        out = {}
        for k, x in s.items():
            if k == "w":
                x = x.clone()
                x[1:nz] = self.mm(faces, x[1:nz].contiguous())
                out[k] = x
            else:
                out[k] = self.mm(m.get(k, None) if k in m else centred(p["kappa"]), x)
        return out

    def divergence(self, u, v, w):
        wz = (w[1:] - w[:-1]) if self.zb else torch.roll(w, -1, 0) - w
        return ((torch.roll(u, -1, 2) - u) / self.dx + (torch.roll(v, -1, 1) - v) / self.dy
                + wz / self.dzc)

    def gradient(self, q):
        gx = (q - torch.roll(q, 1, 2)) / self.dx
        gy = (q - torch.roll(q, 1, 1)) / self.dy
        if not self.zb:
            gz = (q - torch.roll(q, 1, 0)) / self.dzf[:-1]
        else:
            gz = torch.zeros((self.nz + 1,) + q.shape[1:], device=DEV, dtype=torch.float64)
            gz[1:self.nz] = (q[1:] - q[:-1]) / self.dzf[1:self.nz]
        if self.solid is not None:
            gx, gy, gz = (g * o for g, o in zip((gx, gy, gz), self.open))
        return gx, gy, gz

    def project(self, u, v, w):
        """Velocity made divergence-free (the time step drops out)."""
        if self.solid is None:
            q = self.poisson(self.divergence(u, v, w))
        else:
            u, v, w = (a * o for a, o in zip((u, v, w), self.open))
            b = self.divergence(u, v, w) * self.solid
            q, r = torch.zeros_like(b), b.clone()
            z = self.poisson(r) * self.solid
            d, rz, b2 = z.clone(), (r * z).sum(), float(b.square().sum())
            for _ in range(300):
                ad = self.divergence(*self.gradient(d)) * self.solid
                al = rz / (d * ad).sum()
                q += al * d
                r -= al * ad
                if float(r.square().sum()) <= 1e-27 * b2:
                    break
                z = self.poisson(r) * self.solid
                new = (r * z).sum()
                d = z + (new / rz) * d
                rz = new
        gx, gy, gz = self.gradient(q)
        return u - gx, v - gy, w - gz

    def step(self, s, dt, extra=None):
        gam, zet, G0 = (8 / 15, 5 / 12, 3 / 4), (0.0, 17 / 60, 5 / 12), None
        for m in range(3):
            G = self.tendencies(s)
            if extra is not None:
                for k, a in extra(s).items():
                    G[k] = G[k] + a
            s = {k: s[k] + dt * (gam[m] * G[k] - (zet[m] * G0[k] if m else 0.0)) for k in s}
            if self.p.get("implicit_z"):
                s = self.implicit(s, (gam[m] - zet[m]) * dt)
            s["u"], s["v"], s["w"] = self.project(s["u"], s["v"], s["w"])
            G0 = G
        return s


def _exact_step(case, seed):
    p = _params(case)
    box = _Box(p)
    s = {k: a.double() for k, a in _fields(case, p, seed).items()}
    if box.solid is not None:
        for k, o in zip("uvw", box.open):
            s[k] = s[k] * o
    extra = _learned(box, seed) if case["kind"] == "closure" else None
    for _ in range(case["steps"]):
        s = box.step(s, _dt(case), extra)
    return s


def _learned(box, seed):
    """The learned closure's tendencies: the network on the standardised
    5 x 5 x 5 neighbourhoods, then the divergence of its vertical fluxes."""
    net = {k: torch.from_numpy(v).to(DEV).double() for k, v in _network(seed).items()}
    p, nz = box.p, box.nz
    st = torch.tensor(STATS, device=DEV, dtype=torch.float64)

    def tend(s):
        P = [_pad(s["u"], True), _pad(s["v"], True), _pad(s["w"], True, True),
             p["g"] * (p["alpha"] * (_pad(s["T"], True) - p["t_ref"])
                       - p["beta"] * (_pad(s["S"], True) - p["s_ref"]))]
        ys = []
        for k in range(nz):
            rows = []
            for q in range(4):
                a = (P[q] - st[q]) / st[4 + q]
                for dk in range(-2, 3):
                    for dj in range(-2, 3):
                        for di in range(-2, 3):
                            rows.append(a[_H + k + dk, _H + dj:_H + dj + box.ny,
                                          _H + di:_H + di + box.nx].reshape(-1))
            ys.append(_mlp(net, torch.stack(rows, 1)))
        F = torch.stack(ys).reshape(nz, box.ny, box.nx, 4) * st[12:16] + st[8:12]
        tu, tv, tw, jb = (F[..., q] for q in range(4))
        zero = torch.zeros_like(tu[:1])

        def dz(a):
            f = torch.cat([zero, 0.5 * (a[1:] + a[:-1]), zero])
            return -(f[1:] - f[:-1]) / box.dzc
        gw = torch.cat([zero, -(tw[1:] - tw[:-1]) / box.dzf[1:nz], zero])
        return {"u": dz(0.5 * (tu + torch.roll(tu, 1, 2))),
                "v": dz(0.5 * (tv + torch.roll(tv, 1, 1))),
                "T": dz(jb / (p["g"] * p["alpha"])), "w": gw}
    return tend


def _exact_sector(case, seed):
    nx, ny, nz = case["nx"], case["ny"], case["nz"]
    s = {k: a.double() for k, a in _sector_fields(case, seed).items()}
    R, depth, omega, grav = 6.371e6, 3000.0, 7.292115e-5, 9.81
    nu = ka = 1e-4
    dlam, dphi = 2 * math.pi / nx, math.radians(140.0 / ny)
    dz, dy, dt, N = depth / nz, 6.371e6 * math.radians(140.0 / ny), 600.0, case["N"]
    weno, H = _Weno(3), 3
    ar = torch.arange(-4, ny + 6, device=DEV, dtype=torch.float64)
    phf = math.radians(-70.0) + ar * dphi            # faces j = -4 ..
    phc = phf + 0.5 * dphi
    dxc, dxf = R * torch.cos(phc) * dlam, R * torch.cos(phf) * dlam
    area = R * R * dlam * (torch.sin(phf + dphi) - torch.sin(phf))
    acor = R * R * dlam * (torch.sin(phc) - torch.sin(phc - dphi))

    def row(a, j0, j1):
        return a[4 + j0:4 + j1][None, :, None]

    def pad(a, vface=False):
        i = torch.arange(-H, nz + H, device=DEV)
        a = a.index_select(0, torch.where(i < 0, -1 - i, torch.where(i >= nz, 2 * nz - 1 - i, i)))
        i = torch.arange(-H, ny + H, device=DEV)
        if vface:
            sg = torch.where((i < 0) | (i > ny), -1.0, 1.0).double()
            sg[(i == 0) | (i == ny)] = 0.0
            a = a.index_select(1, torch.where(i < 0, -i, torch.where(i > ny, 2 * ny - i, i)))
            a = a * sg[None, :, None]
        else:
            a = a.index_select(1, torch.where(i < 0, -1 - i,
                                              torch.where(i >= ny, 2 * ny - 1 - i, i)))
        return a.index_select(2, torch.arange(-H, nx + H, device=DEV) % nx)

    def blk(P, j0, j1, i0, i1):
        return P[H:H + nz, H + j0:H + j1, H + i0:H + i1]

    def vflux(col, W):
        f = W * weno([col[H + o:H + o + nz + 1] for o in range(-3, 3)], W)
        f[0] = 0.0
        f[nz] = W[nz] * col[H + nz - 1]
        return f

    def tend(s):
        up, vp = pad(s["u"]), pad(s["v"], True)
        fx = dy * (blk(up, 0, ny, 0, nx + 1) - blk(up, 0, ny, -1, nx))
        fy = (row(dxf, 1, ny + 1) * blk(vp, 1, ny + 1, -1, nx)
              - row(dxf, 0, ny) * blk(vp, 0, ny, -1, nx))
        div = (fx + fy) / row(area, 0, ny)
        w = torch.cat([torch.zeros_like(div[:1]), -dz * torch.cumsum(div, 0)])  # columns -1..
        wc = w[:, :, 1:]
        b = grav * (2e-4 * s["T"] - 8e-4 * (s["S"] - 35.0))
        half = torch.cat([0.5 * (b[1:] + b[:-1]), 0.5 * b[-1:]])
        pp = pad(-dz * torch.flip(torch.cumsum(torch.flip(half, (0,)), 0), (0,)))
        j0, j1, i0, i1 = -2, ny + 3, -2, nx + 3
        zeta = (dy * (blk(vp, j0, j1, i0, i1) - blk(vp, j0, j1, i0 - 1, i1 - 1))
                - (row(dxc, j0, j1) * blk(up, j0, j1, i0, i1)
                   - row(dxc, j0 - 1, j1 - 1) * blk(up, j0 - 1, j1 - 1, i0, i1))) \
            / row(acor, j0, j1)

        def Z(a, b, c, d):
            return zeta[:, a + 2:b + 2, c + 2:d + 2]
        ke = 0.25 * (blk(up, -1, ny + 1, -1, nx + 1) ** 2 + blk(up, -1, ny + 1, 0, nx + 2) ** 2
                     + blk(vp, -1, ny + 1, -1, nx + 1) ** 2 + blk(vp, 0, ny + 2, -1, nx + 1) ** 2)
        G = {}
        u = s["u"]
        vb = 0.25 * (blk(vp, 0, ny, -1, nx - 1) + blk(vp, 0, ny, 0, nx)
                     + blk(vp, 1, ny + 1, -1, nx - 1) + blk(vp, 1, ny + 1, 0, nx))
        g = weno([Z(o, ny + o, 0, nx) for o in range(-2, 4)], vb) * vb
        g = g + 2 * omega * torch.sin(row(phc, 0, ny)) * vb
        g = g - (ke[:, 1:-1, 1:-1] - ke[:, 1:-1, :-2]) / row(dxc, 0, ny)
        g = g - (blk(pp, 0, ny, 0, nx) - blk(pp, 0, ny, -1, nx - 1)) / row(dxc, 0, ny)
        W = 0.5 * (w[:, :, :nx] + w[:, :, 1:])
        f = vflux(up[:, H:H + ny, H:H + nx], W)
        g = g - (f[1:] - f[:-1]) / dz + u * (W[1:] - W[:-1]) / dz
        f = torch.cat([torch.zeros_like(u[:1]), nu * (u[1:] - u[:-1]) / dz, s["tau_x"]])
        G["u"] = g + (f[1:] - f[:-1]) / dz
        v = blk(vp, 0, ny + 1, 0, nx)
        ub = 0.25 * (blk(up, -1, ny, 0, nx) + blk(up, -1, ny, 1, nx + 1)
                     + blk(up, 0, ny + 1, 0, nx) + blk(up, 0, ny + 1, 1, nx + 1))
        g = -weno([Z(0, ny + 1, o, nx + o) for o in range(-2, 4)], ub) * ub
        g = g - 2 * omega * torch.sin(row(phf, 0, ny + 1)) * ub
        g = g - (ke[:, 1:, 1:-1] - ke[:, :-1, 1:-1]) / dy
        g = g - (blk(pp, 0, ny + 1, 0, nx) - blk(pp, -1, ny, 0, nx)) / dy
        wp = torch.zeros((nz + 1, ny + 2, nx), device=DEV, dtype=torch.float64)
        wp[:, 1:ny + 1] = wc
        W = 0.5 * (wp[:, :-1] + wp[:, 1:])
        f = vflux(vp[:, H:H + ny + 1, H:H + nx], W)
        g = g - (f[1:] - f[:-1]) / dz + v * (W[1:] - W[:-1]) / dz
        f = torch.cat([torch.zeros_like(v[:1]), nu * (v[1:] - v[:-1]) / dz, s["tau_y"]])
        g = g + (f[1:] - f[:-1]) / dz
        g[:, 0] = 0.0
        g[:, ny] = 0.0
        G["v"] = g
        uf = blk(up, 0, ny, 0, nx + 1)
        az = row(area, 0, ny)
        for n in ("T", "S"):
            c, cp = s[n], pad(s[n])
            fx = uf * weno([blk(cp, 0, ny, o, nx + 1 + o) for o in range(-3, 3)], uf) * (dy * dz)
            fy = v * weno([blk(cp, o, ny + 1 + o, 0, nx) for o in range(-3, 3)], v) \
                * row(dxf, 0, ny + 1) * dz
            fy[:, 0] = 0.0
            fy[:, ny] = 0.0
            fz = vflux(cp[:, H:H + ny, H:H + nx], wc) * az
            fz[1:nz] -= ka * (c[1:] - c[:-1]) / dz * az
            G[n] = -((fx[:, :, 1:] - fx[:, :, :-1]) + (fy[:, 1:] - fy[:, :-1])
                     + (fz[1:] - fz[:-1])) / (az * dz)
        return G

    n = np.arange(1, 2 * N)
    wt = np.cos(0.5 * np.pi * (n - N) / N) ** 2
    wt = wt / wt.sum()
    eta, U, V = s["eta"][0], s["U"][0], s["V"][0]
    G0 = None
    lf, ac, dxu = row(dxf, 0, ny + 1)[0], row(area, 0, ny)[0], row(dxc, 0, ny)[0]
    for _ in range(case["steps"]):
        G = tend(s)
        comb = {k: (1.6 * G[k] - 0.6 * G0[k]) if G0 is not None else G[k] for k in G}
        for k in G:
            s[k] = s[k] + dt * comb[k]
        GU, GV = dz * comb["u"].sum(0), dz * comb["v"].sum(0)
        eb, ub, vb = torch.zeros_like(eta), torch.zeros_like(U), torch.zeros_like(V)
        tau = dt / N
        for a in wt:
            fy = lf * V
            eta = eta - tau * (dy * (torch.roll(U, -1, 1) - U) + fy[1:] - fy[:-1]) / ac
            U = U - tau * (grav * depth * (eta - torch.roll(eta, 1, 1)) / dxu - GU)
            V = V.clone()
            V[1:-1] -= tau * (grav * depth * (eta[1:] - eta[:-1]) / dy - GV[1:-1])
            eb += a * eta
            ub += a * U
            vb += a * V
        eta, U, V = eb, ub, vb
        s["u"] = s["u"] + ((U - dz * s["u"].sum(0)) / depth)[None]
        s["v"] = s["v"] + ((V - dz * s["v"].sum(0)) / depth)[None]
        s["v"][:, 0] = 0.0
        s["v"][:, ny] = 0.0
        G0 = G
    return {k: s[k] for k in ("u", "v", "T", "S")}
