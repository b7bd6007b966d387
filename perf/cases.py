"""The work users of this framework have it do, as measurable cases.

Five kinds of call, each through the public entry points of the package:

* ``step``         a coupled run advanced by an even number of steps
                   (``Solver.step``), 2D (D2Q9) and 3D (D3Q19), both element
                   types, every flux scheme, with and without the second
                   scalar, size classes, and the full force and settling;
* ``sweep``        a batch of uneven 2D runs advanced together;
* ``gradient``     ``DepositedMass``: forward and backward of the deposited
                   mass, 2D and 3D;
* ``diagnostics``  what a program reads between steps: masses, the front
                   height, its spectra.

The fields are those of a run under way: a particle-laden upper layer over a
dilute lower one, an interface bent by a few modes and roughened by noise, and
a smooth flow of about 1e-2 in lattice units.  Workloads the package holds a
tuned launch for use it, every other size runs as a program that sets no
launch shape does.  Runs in single precision hand their deposit counters
(FP64 sums of single-precision values) and objective back in the precision of
the run.
"""
import math
import random

import torch
from torch.utils.checkpoint import checkpoint

from paper_2106_07694_amd import adjoint, autotune, lbw

DEV = "cuda"
EPS = 1e-6                      # WENO regularisation (the package's default)
SWEEP_GRIDS = ((128, 256), (256, 512), (512, 1024))

# ---------------------------------------------------------------------------
# the cases
# ---------------------------------------------------------------------------


def _step(nx, ny, nz, precision, steps, **more):
    c = dict(kind="step", nx=nx, ny=ny, nz=nz, precision=precision, steps=steps, scheme="weno5",
             sugar=False, full_force=False, classes=1, periodic=False, tuned="")
    c.update(more)
    return c


def listed():
    return [
        # the small validation run of the test-suite and the smoke test: one
        # launch-bound run a user iterates on, in double precision
        dict(_step(64, 128, 1, "fp64", 100), name="step_2d_fp64_64x128"),
        # the two-scalar 2D production run, with its tuned launch
        dict(_step(1024, 2048, 1, "fp32_shifted", 20, sugar=True, tuned="2d_fp32_shifted_s_1024x2048"),
             name="step_2d_sugar_1024x2048"),
        # the paper's full force and settling on a grid that is no power of
        # two and that nobody tuned
        dict(_step(515, 1030, 1, "fp32_shifted", 20, sugar=True, full_force=True),
             name="step_2d_full_force_515x1030"),
        # the paper's own third-order scheme in double precision
        dict(_step(256, 512, 1, "fp64", 20, scheme="weno3"), name="step_2d_fp64_weno3_256x512"),
        # the flagship 3D run, with its tuned launch
        dict(_step(256, 256, 512, "fp32_shifted", 10, tuned="3d_d3q19_fp32_256x256x512"),
             name="step_3d_256x256x512"),
        # a small exploratory 3D run on a ragged grid
        dict(_step(97, 63, 130, "fp32_shifted", 20), name="step_3d_97x63x130"),
        # a 3D reference run in double precision
        dict(_step(128, 96, 160, "fp64", 10), name="step_3d_fp64_128x96x160"),
        # particle size classes in 3D
        dict(_step(128, 128, 192, "fp32_shifted", 10, classes=4), name="step_3d_4_classes_128x128x192"),
        # a parameter sweep, batched and graph-replayed as tuned
        dict(kind="sweep", runs=30, plan=1003, steps=20, tuned="sweep_64", name="sweep_30"),
        # the gradient of the deposited mass on the adjoint workload
        dict(kind="gradient", nx=512, ny=1024, nz=1, precision="fp32_shifted", steps=100,
             tuned="2d_fp32_adjoint_512x1024", name="gradient_2d_512x1024"),
        # the same in 3D
        dict(kind="gradient", nx=64, ny=48, nz=96, precision="fp32_shifted", steps=20, tuned="",
             name="gradient_3d_64x48x96"),
        # the diagnostics of the flagship run
        dict(kind="diagnostics", nx=256, ny=256, nz=512, precision="fp32_shifted",
             name="diagnostics_3d_256x256x512"),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["step", "step", "step", "step", "sweep", "gradient", "gradient", "diagnostics"])
    three = rng.random() < 0.5
    precision = rng.choice(["fp32_shifted", "fp32_shifted", "fp32_shifted", "fp64", "fp64_shifted"])
    if kind == "sweep":
        return dict(kind="sweep", runs=rng.randint(2, 30), plan=rng.randrange(1 << 20), steps=2 * rng.randint(4, 10),
                    tuned=rng.choice(["sweep_64", ""]))
    if kind == "gradient":
        nx, ny, nz = ((_log_int(rng, 16, 64), _log_int(rng, 16, 64), _log_int(rng, 24, 96)) if three
                      else (_log_int(rng, 32, 512), _log_int(rng, 48, 1024), 1))
        return dict(kind="gradient", nx=nx, ny=ny, nz=nz, precision=precision, tuned="",
                    steps=rng.randint(8, 20) if three else rng.randint(16, 100))
    if kind == "diagnostics":
        nx, ny, nz = ((_log_int(rng, 24, 256), _log_int(rng, 24, 256), _log_int(rng, 32, 512)) if three
                      else (_log_int(rng, 48, 1024), _log_int(rng, 64, 2048), 1))
        return dict(kind="diagnostics", nx=nx, ny=ny, nz=nz, precision=precision)
    wide = precision != "fp32_shifted"
    if three:
        nx, ny, nz = (_log_int(rng, 16, 160 if wide else 256), _log_int(rng, 16, 160 if wide else 256),
                      _log_int(rng, 24, 200 if wide else 400))
    else:
        nx, ny, nz = _log_int(rng, 32, 1024), _log_int(rng, 48, 2048), 1
    sugar = rng.random() < 0.4
    return _step(nx, ny, nz, precision, 2 * rng.randint(4, 5 if three else 20),
                 scheme=rng.choice(["weno5", "weno5", "weno5", "weno5", "weno3", "upwind1"]), sugar=sugar,
                 full_force=sugar and rng.random() < 0.4,
                 classes=rng.randint(2, 4) if rng.random() < 0.2 else 1, periodic=rng.random() < 0.15)


# ---------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------

# D2Q9 and D3Q19 in the order include/lbw.h fixes
_C9 = [(0, 0, 0), (1, 0, 0), (0, 1, 0), (-1, 0, 0), (0, -1, 0), (1, 1, 0), (-1, 1, 0), (-1, -1, 0), (1, -1, 0)]
_W9 = [4 / 9] + [1 / 9] * 4 + [1 / 36] * 4
_C19 = [(0, 0, 0), (1, 0, 0), (-1, 0, 0), (0, 1, 0), (0, -1, 0), (0, 0, 1), (0, 0, -1),
        (1, 1, 0), (-1, -1, 0), (1, -1, 0), (-1, 1, 0), (1, 0, 1), (-1, 0, -1), (1, 0, -1), (-1, 0, 1),
        (0, 1, 1), (0, -1, -1), (0, 1, -1), (0, -1, 1)]
_W19 = [1 / 3] + [1 / 18] * 6 + [1 / 36] * 12


def _physics(case, run=None):
    """The parameters of a case (the package's workloads' values), as the
    keyword arguments of RunConfig."""
    three = case.get("nz", 1) > 1
    classes = case.get("classes", 1)
    p = dict(lattice=lbw.D3Q19 if three else lbw.D2Q9, precision=case.get("precision", "fp32_shifted"),
             nx=case.get("nx"), ny=case.get("ny"), nz=case.get("nz", 1), tau=0.55 if three else 0.6,
             vs=5e-4 if three else 1e-3, kappa_c=5e-4 if three else 1e-3, gp_c=1e-5,
             scheme_c=case.get("scheme", "weno5"), vert_periodic=case.get("periodic", False),
             has_s=case.get("sugar", False), weno_eps=EPS)
    if p["has_s"]:
        p.update(kappa_s=1e-4, gp_s=2e-5, vs=5e-4)
    if case.get("full_force", False):
        p.update(vs_s=0.5, phi_c=1e-3)
    if classes > 1:
        p.update(n_classes=classes, vs_class=tuple(2.5e-4 * (i + 1) for i in range(classes)),
                 kappa_class=(p["kappa_c"],) * classes, vs=0.0, kappa_c=0.0)
    if run is not None:
        p.update(run)
    return p


def _dtype(p):
    return torch.float32 if p["precision"] == "fp32_shifted" else torch.float64


def _fields(p, seed, c0=1.0):
    """C, S (or None) and the velocity of a run under way, in the run's type."""
    g = torch.Generator(device=DEV).manual_seed(int(seed) * 7919 + 17)
    three = p["nz"] > 1
    nx, ny, nz = p["nx"], p["ny"], p["nz"]
    shape, nv = (nz, ny, nx), (nz if three else ny)
    ax = lambda n, d: torch.arange(n, device=DEV, dtype=torch.float64).reshape([-1 if i == d else 1 for i in range(3)])  # noqa: E731
    x, y, z = ax(nx, 2), ax(ny, 1), ax(nz, 0)
    v = z if three else y
    r = torch.rand(8, generator=g, device=DEV, dtype=torch.float64).tolist()
    m = 1 + int(3 * r[0])
    px = 2 * math.pi * (m * x / nx + r[1])
    py = 2 * math.pi * (y / ny + r[2]) if three else torch.zeros_like(px)
    level = 0.5 * (nv - 1) + 2.5 * torch.cos(px + (r[3] * 6.0 if three else 0.0)) * torch.cos(0.5 * py)
    layer = 0.5 * (1 + torch.tanh((v - level) / 2.0))
    n = max(1, p.get("n_classes", 1))
    cshape = shape if n == 1 else (n,) + shape
    noise = torch.rand(cshape, generator=g, device=DEV, dtype=_dtype(p))
    c = (c0 / n) * (0.05 + 0.95 * layer) + (1e-3 / n) * (2 * noise.double() - 1)
    s = ((1 - layer) + torch.zeros(shape, device=DEV, dtype=torch.float64)) if p["has_s"] else None
    up = math.pi * (v + 0.5) / nv
    a = 8e-3 * (0.75 + 0.5 * r[4])
    u = [a * torch.sin(px) * torch.cos(up) * torch.cos(py), a * torch.cos(px) * torch.sin(up)]
    if three:
        u = [u[0], 0.7 * a * torch.sin(py) * torch.cos(up) * torch.cos(px), u[1] * torch.cos(py)]
    u = torch.stack([t + torch.zeros(shape, device=DEV, dtype=torch.float64) for t in u])
    cast = lambda t: None if t is None else t.to(_dtype(p)).contiguous()  # noqa: E731
    return cast(c), cast(s), cast(u)


def _sweep_plan(case):
    r = random.Random(case["plan"])
    runs = []
    for _ in range(case["runs"]):
        nx, ny = r.choice(SWEEP_GRIDS)
        c0 = r.uniform(0.25, 4.0)
        vs = math.exp(r.uniform(math.log(1e-4), math.log(2e-3)))
        runs.append((c0, _physics(case, dict(nx=nx, ny=ny, vs=vs))))
    return runs


def _launch(case):
    return (autotune.lookup(case["tuned"]) or {}) if case["tuned"] else {}


def _fill(sol, p, seed, run=0, c0=1.0):
    c, s, u = _fields(p, seed, c0)
    sol.set_field("c", c, run)
    if s is not None:
        sol.set_field("s", s, run)
    sol.init_equilibrium(run, u=u)


def _equilibrium(p, u):
    """Populations f_i (not shifted) at density 1 and velocity u, FP64."""
    cs, ws = (_C19, _W19) if p["nz"] > 1 else (_C9, _W9)
    u = u.double()
    usq = (u * u).sum(0)
    f = []
    for c, w in zip(cs, ws):
        cu = sum(c[d] * u[d] for d in range(u.shape[0]))
        f.append(w * (1 + 3 * cu + 4.5 * cu * cu - 1.5 * usq))
    return torch.stack([t + torch.zeros_like(usq) for t in f])


def _weights(p, like):
    ws = _W19 if p["nz"] > 1 else _W9
    return torch.tensor(ws, dtype=torch.float64, device=DEV).reshape([-1] + [1] * (like.dim() - 1))


def _shifted(p):
    return p["precision"] != "fp64"


def _gradient_inputs(case, seed):
    p = _physics(case)
    c, _, u = _fields(p, seed)
    f = _equilibrium(p, u)
    f0 = ((f - _weights(p, f)) if _shifted(p) else f).to(_dtype(p)).contiguous()
    return p, c, f0, torch.tensor(p["vs"], dtype=_dtype(p), device=DEV)


# ---------------------------------------------------------------------------
# the calls
# ---------------------------------------------------------------------------


def prepare(case, seed):
    kind = case["kind"]
    if kind == "gradient":
        p, c, f0, vs = _gradient_inputs(case, seed)
        return dict(kind=kind, cfg=lbw.RunConfig(**p), c=c, f0=f0, vs=vs, steps=case["steps"],
                    launch=_launch(case) or None)
    if kind == "sweep":
        plan = _sweep_plan(case)
        stream = torch.cuda.Stream()
        sol = lbw.Solver([lbw.RunConfig(**p) for _, p in plan], stream=stream)
        sol.set_launch(**_launch(case))
        torch.cuda.synchronize()
        for i, (c0, p) in enumerate(plan):
            _fill(sol, p, seed * 100 + i, i, c0)
        return dict(kind=kind, sol=sol, steps=case["steps"])
    p = _physics(case)
    sol = lbw.Solver(lbw.RunConfig(**p))
    sol.set_launch(**(_launch(case) if kind == "step" else {}))
    _fill(sol, p, seed)
    if kind == "diagnostics":
        return dict(kind=kind, sol=sol, cfg=sol.cfgs[0], plane=(p["nz"] if p["nz"] > 1 else p["ny"]) // 2)
    return dict(kind=kind, sol=sol, steps=case["steps"], dtype=_dtype(p))


def run(state):
    kind = state["kind"]
    if kind == "gradient":
        c0 = state["c"].detach().requires_grad_()
        vs = state["vs"].detach().requires_grad_()
        mass = adjoint.DepositedMass.apply(c0, vs, state["cfg"], state["steps"], None, state["launch"], state["f0"])
        mass.backward()
        return dict(mass=mass.detach().to(c0.dtype), c=c0.grad, vs=vs.grad)
    sol = state["sol"]
    if kind == "diagnostics":
        three = state["cfg"].dim == 3
        out = dict(mass=sol.reduce(lbw.MASS_C), fluid=sol.reduce(lbw.MASS_FLUID), deposit=sol.reduce(lbw.DEPOSIT),
                   below=sol.mass_below(state["plane"]), front=sol.front_height(0.5))
        out["psd_x"] = sol.front_psd(out["front"], 0, -1 if three else 0)
        if three:
            out["psd_y"] = sol.front_psd(out["front"], 1, -1)
        return out
    sol.step(state["steps"])
    # an even number of steps later the fields are in the caller's own buffers
    if kind == "sweep":
        with torch.cuda.stream(sol.stream):
            deposit = torch.cat([t["deposit"] for t in sol.tensors]).float()
        return dict(deposit=deposit, c=[t["c"] for t in sol.tensors], f=[t["f"] for t in sol.tensors])
    t = sol.tensors[0]
    out = dict(f=t["f"], c=t["c"], u=t["u"], deposit=t["deposit"].to(state["dtype"]))
    if t["s"] is not None:
        out["s"] = t["s"]
    return out


# ---------------------------------------------------------------------------
# what a pass cannot do without
# ---------------------------------------------------------------------------


def _step_work(p):
    """Bytes and operations of one step of one run: the state (populations and
    scalars) read once and written once; per cell about 23 operations a
    population for moments and collision, and per face of each of the three
    Runge-Kutta stages one reconstruction, two per cell and axis being shared."""
    cells, dim = p["nx"] * p["ny"] * p["nz"], 3 if p["nz"] > 1 else 2
    q, n = (19 if dim == 3 else 9), max(1, p.get("n_classes", 1))
    size = 4 if p["precision"] == "fp32_shifted" else 8
    face = {"weno5": 70, "weno3": 32, "upwind1": 8}[p["scheme_c"]]
    return (2 * size * cells * (q + n + (1 if p["has_s"] else 0)),
            cells * (23 * q + 3 * n * dim * face + (8 * dim if p["has_s"] else 0)))


def work(case):
    kind = case["kind"]
    if kind == "sweep":
        per = [_step_work(p) for _, p in _sweep_plan(case)]
        return dict(bytes=case["steps"] * sum(b for b, _ in per), flops=case["steps"] * sum(f for _, f in per))
    p = _physics(case)
    cells = p["nx"] * p["ny"] * p["nz"]
    size = 4 if p["precision"] == "fp32_shifted" else 8
    if kind == "diagnostics":
        # C for the sums (once whole, half again below the plane), for the
        # front up to it, and the populations for the fluid mass
        q = 19 if p["nz"] > 1 else 9
        return dict(bytes=size * cells * (q + 2), flops=cells * (q + 3))
    b, f = _step_work(p)
    if kind == "gradient":
        # forward, the replay of each segment, and the reverse steps: the
        # adjoint state read and written, the moments and stages read, and
        # about three times the operations of the forward step
        dim = 3 if p["nz"] > 1 else 2
        return dict(bytes=case["steps"] * (3 * b + size * cells * (dim + 4)), flops=case["steps"] * 5 * f)
    return dict(bytes=case["steps"] * b, flops=case["steps"] * f)


# ---------------------------------------------------------------------------
# the same calls in 64 bits, in plain torch
# ---------------------------------------------------------------------------


def _cut(t, dim, lo, hi):
    return t.narrow(dim, lo, hi - lo)


def _extended(t, dim, walls, odd=False):
    """t with three more cells at both ends of an axis."""
    n = t.shape[dim]
    if walls:
        lo, hi = _cut(t, dim, 0, 3).flip(dim), _cut(t, dim, n - 3, n).flip(dim)
        return torch.cat([-lo, t, -hi] if odd else [lo, t, hi], dim)
    return torch.cat([_cut(t, dim, n - 3, n), t, _cut(t, dim, 0, 3)], dim)


def _weno5(h, a):
    q0 = (2 * h[0] - 7 * h[1] + 11 * h[2]) / 6
    q1 = (-h[1] + 5 * h[2] + 2 * h[3]) / 6
    q2 = (2 * h[2] + 5 * h[3] - h[4]) / 6
    b0 = 13 / 12 * (a[0] - 2 * a[1] + a[2]) ** 2 + (a[0] - 4 * a[1] + 3 * a[2]) ** 2 / 4
    b1 = 13 / 12 * (a[1] - 2 * a[2] + a[3]) ** 2 + (a[1] - a[3]) ** 2 / 4
    b2 = 13 / 12 * (a[2] - 2 * a[3] + a[4]) ** 2 + (3 * a[2] - 4 * a[3] + a[4]) ** 2 / 4
    w0, w1, w2 = 0.1 / (EPS + b0) ** 2, 0.6 / (EPS + b1) ** 2, 0.3 / (EPS + b2) ** 2
    return (w0 * q0 + w1 * q1 + w2 * q2) / (w0 + w1 + w2)


def _weno3(h, a):
    qu, qc = (3 * h[1] - h[0]) / 2, (h[1] + h[2]) / 2
    wu, wc = 1 / (3 * (EPS + (a[1] - a[0]) ** 2) ** 2), 2 / (3 * (EPS + (a[2] - a[1]) ** 2) ** 2)
    return (wu * qu + wc * qc) / (wu + wc)


def _face_fluxes(a, w, dim, kappa, scheme):
    """Fluxes through the n + 1 faces of an axis extended by three cells."""
    n = a.shape[dim] - 6
    A = [_cut(a, dim, i, i + n + 1) for i in range(6)]
    W = [_cut(w, dim, i, i + n + 1) for i in range(6)]
    pos = (W[2] + W[3]) >= 0
    up = lambda t, i: torch.where(pos, t[i], t[5 - i])  # noqa: E731
    if scheme == "upwind1":
        h = up(W, 2) * up(A, 2)
    else:
        at = range(5) if scheme == "weno5" else range(1, 4)
        aa = [up(A, i) for i in at]
        hh = [up(W, i) * t for i, t in zip(at, aa)]
        h = _weno5(hh, aa) if scheme == "weno5" else _weno3(hh, aa)
    return h - kappa * (A[3] - A[2])


def _rhs(p, a, u, fall, kappa):
    """-div of the fluxes of a; fall: settling speed (number or field)."""
    dims = 3 if p["nz"] > 1 else 2
    out = 0
    for d in range(dims):
        dim, vert = 2 - d, d == dims - 1
        walls = vert and not p["vert_periodic"]
        w = _extended(u[d], dim, walls, odd=walls)
        if vert:
            w = w - (_extended(fall, dim, walls) if torch.is_tensor(fall) and fall.dim() == 3 else fall)
        fl = _face_fluxes(_extended(a, dim, walls), w, dim, kappa, p["scheme_c"])
        if walls:
            n = a.shape[dim]
            low = _cut(fall, dim, 0, 1) if torch.is_tensor(fall) and fall.dim() == 3 else fall
            fl = torch.cat([-low * _cut(a, dim, 0, 1), _cut(fl, dim, 1, n), torch.zeros_like(_cut(a, dim, 0, 1))], dim)
        out = out - (_cut(fl, dim, 1, fl.shape[dim]) - _cut(fl, dim, 0, fl.shape[dim] - 1))
    return out


def _sugar(p, s, u):
    dims = 3 if p["nz"] > 1 else 2
    out = s
    for d in range(dims):
        dim, n = 2 - d, s.shape[2 - d]
        walls = d == dims - 1 and not p["vert_periodic"]
        ends = lambda t: torch.cat([_cut(t, dim, n - 1, n), t, _cut(t, dim, 0, 1)], dim)  # noqa: E731, B023
        a, w = ends(s), ends(u[d])
        a0, a1, w0, w1 = _cut(a, dim, 0, n + 1), _cut(a, dim, 1, n + 2), _cut(w, dim, 0, n + 1), _cut(w, dim, 1, n + 2)
        fl = torch.where(w0 + w1 >= 0, w0 * a0, w1 * a1) - p["kappa_s"] * (a1 - a0)
        if walls:
            none = torch.zeros_like(_cut(fl, dim, 0, 1))
            fl = torch.cat([none, _cut(fl, dim, 1, n), none], dim)
        out = out - (_cut(fl, dim, 1, n + 1) - _cut(fl, dim, 0, n))
    return out


def _advance(p, f, c, s, dep, vs):
    """One coupled step: populations f (not shifted), a list of concentrations
    c with their settling speeds vs, S, a list of deposits."""
    three = p["nz"] > 1
    dims = 3 if three else 2
    cs, ws = (_C19, _W19) if three else (_C9, _W9)
    up_dim = 0 if three else 1                       # vertical axis of a (nz, ny, nx) field
    total = sum(c)
    force = -p["gp_c"] * total
    if s is not None:
        force = force - p["gp_s"] * s * (1 - p.get("phi_c", 0.0) * total)
    rho = f.sum(0)
    u = []
    for d in range(dims):
        m = sum(v[d] * f[i] for i, v in enumerate(cs) if v[d])
        u.append((m + (force / 2 if d == dims - 1 else 0)) / rho)
    usq, uf = sum(t * t for t in u), u[-1] * force
    post = []
    for i, (v, w) in enumerate(zip(cs, ws)):
        cu = sum(v[d] * u[d] for d in range(dims))
        eq = w * rho * (1 + 3 * cu + 4.5 * cu * cu - 1.5 * usq)
        cf = v[dims - 1] * force
        post.append(f[i] - (f[i] - eq) / p["tau"] + (1 - 0.5 / p["tau"]) * w * (3 * (cf - uf) + 9 * cu * cf))
    new = []
    for i, v in enumerate(cs):
        t = torch.roll(post[i], shifts=(v[2], v[1], v[0]), dims=(0, 1, 2))
        rise = v[dims - 1]
        if rise and not p["vert_periodic"]:
            back = post[cs.index((-v[0], -v[1], -v[2]))]
            n = t.shape[up_dim]
            if rise > 0:
                t = torch.cat([_cut(back, up_dim, 0, 1), _cut(t, up_dim, 1, n)], up_dim)
            else:
                t = torch.cat([_cut(t, up_dim, 0, n - 1), _cut(back, up_dim, n - 1, n)], up_dim)
        new.append(t)
    c_new, dep_new = [], []
    kappas = p["kappa_class"] if len(c) > 1 else (p["kappa_c"],)
    for a, k, speed, d0 in zip(c, kappas, vs, dep):
        fall = speed * (1 - p["vs_s"] * s) if p.get("vs_s", 0.0) else speed
        a1 = a + _rhs(p, a, u, fall, k)
        a2 = 0.75 * a + 0.25 * (a1 + _rhs(p, a1, u, fall, k))
        c_new.append(a / 3 + 2 / 3 * (a2 + _rhs(p, a2, u, fall, k)))
        if not p["vert_periodic"]:
            low = _cut(fall, up_dim, 0, 1) if torch.is_tensor(fall) and fall.dim() == 3 else fall
            a, a1, a2 = (_cut(t, up_dim, 0, 1) for t in (a, a1, a2))
            d0 = d0 + (low * (a / 6 + a1 / 6 + 2 / 3 * a2)).reshape(-1)
        dep_new.append(d0)
    return torch.stack(new), c_new, (None if s is None else _sugar(p, s, u)), dep_new, torch.stack(u)


def _exact_run(p, seed, steps, c0=1.0):
    c, s, u = _fields(p, seed, c0)
    n = max(1, p.get("n_classes", 1))
    f, c, s = _equilibrium(p, u), c.double(), (None if s is None else s.double())
    c = [c] if n == 1 else list(c)
    cols = p["nx"] * (p["ny"] if p["nz"] > 1 else 1)
    dep = [torch.zeros(cols, dtype=torch.float64, device=DEV) for _ in range(n)]
    vs = [p["vs"]] if n == 1 else p["vs_class"]
    for _ in range(steps):
        f, c, s, dep, u = _advance(p, f, c, s, dep, vs)
    f = f - _weights(p, f) if _shifted(p) else f
    one = lambda t: t[0] if n == 1 else torch.stack(t)  # noqa: E731
    return dict(f=f, c=one(c), u=u, deposit=one(dep), s=s)


def _exact_gradient(case, seed):
    p, c, f0, vs = _gradient_inputs(case, seed)
    f = f0.double() + (_weights(p, f0) if _shifted(p) else 0)
    c0, v = c.double().requires_grad_(), vs.double().requires_grad_()
    dep = torch.zeros(p["nx"] * (p["ny"] if p["nz"] > 1 else 1), dtype=torch.float64, device=DEV)

    def several(f, c, dep, v, n):
        for _ in range(n):
            f, cl, _, dl, _ = _advance(p, f, [c], None, [dep], [v])
            c, dep = cl[0], dl[0]
        return f, c, dep

    cl, left = c0, case["steps"]
    while left:
        n = min(left, 4)
        f, cl, dep = checkpoint(several, f, cl, dep, v, n, use_reentrant=False)
        left -= n
    mass = dep.sum()
    mass.backward()
    return dict(mass=mass.detach(), c=c0.grad, vs=v.grad)


def _exact_diagnostics(case, seed):
    p = _physics(case)
    c, _, u = _fields(p, seed)
    c, three = c.double(), p["nz"] > 1
    layers = c if three else c.reshape(p["ny"], 1, p["nx"])       # vertical axis first
    nv = layers.shape[0]
    hit = layers >= 0.5
    first = torch.where(hit.any(0), hit.to(torch.uint8).argmax(0), nv)
    hi = layers.gather(0, first.clamp(max=nv - 1)[None])[0]
    lo = layers.gather(0, (first - 1).clamp(min=0)[None])[0]
    front = first - 0.5 + (0.5 - lo) / (hi - lo)
    front = torch.where(first == 0, torch.zeros_like(front), torch.where(first == nv, torch.full_like(front, nv), front))
    psd = lambda h: (torch.fft.rfft(h, dim=-1).abs() ** 2 / h.shape[-1]).mean(0)  # noqa: E731
    whole = lambda t: t.reshape(1).cpu().numpy()  # noqa: E731
    out = dict(mass=whole(c.sum()), fluid=whole(_equilibrium(p, u).sum()), deposit=whole(c.new_zeros(())),
               below=whole(layers[: nv // 2].sum()), front=front if three else front.reshape(-1), psd_x=psd(front))
    if three:
        out["psd_y"] = psd(front.t().contiguous())
    return out


def exact(case, seed):
    kind = case["kind"]
    if kind == "gradient":
        return _exact_gradient(case, seed)
    with torch.no_grad():
        if kind == "diagnostics":
            return _exact_diagnostics(case, seed)
        if kind == "sweep":
            got = [_exact_run(p, seed * 100 + i, case["steps"], c0) for i, (c0, p) in enumerate(_sweep_plan(case))]
            return dict(deposit=torch.cat([g["deposit"] for g in got]), c=[g["c"] for g in got], f=[g["f"] for g in got])
        got = _exact_run(_physics(case), seed, case["steps"])
        if got["s"] is None:
            del got["s"]
        return got
