"""Runs that set no launch shape: the tile and vertical chunk are chosen from
the grid's size, and every choice computes the same values.

The sizes sit where the choice changes (one-plane chunks, chunks that do not
divide the height, tiles wider than the grid, padded tiles, both 3D tile
shapes).  A stage's value at a cell does not depend on the tile or chunk it
was computed in, so the fields equal those of an explicit shape bit for bit.
"""
import numpy as np
import pytest
import torch

from paper_2106_07694_amd import lbw

pytestmark = pytest.mark.gpu

SIZES = {2: [(1, 6, 1), (65, 33, 1), (200, 301, 1), (515, 130, 1), (512, 640, 1)],
         3: [(1, 1, 6), (16, 9, 25), (97, 20, 31), (70, 40, 40), (130, 24, 90)]}


def _fields(cfg, seed):
    rng = np.random.default_rng(seed)
    c = rng.uniform(0.2, 1.0, cfg.shape)
    s = rng.uniform(0.0, 1.0, cfg.shape) if cfg.has_s else None
    return c, s, 0.02 * rng.standard_normal((cfg.dim,) + cfg.shape)


def _run(cfg, fields, launch, steps=3):
    sol = lbw.Solver(cfg)
    sol.set_launch(**launch)
    c, s, u = fields
    sol.set_field("c", c)
    if s is not None:
        sol.set_field("s", s)
    sol.init_equilibrium(u=u)
    sol.step(steps)
    names = ["f", "c", "u", "deposit", "stage1", "stage2"] + (["s"] if s is not None else [])
    out = {n: sol.field(n).clone() for n in names}
    sol.close()
    return out


@pytest.mark.parametrize("precision", ["fp32_shifted", "fp64"])
@pytest.mark.parametrize("dim,size", [(d, s) for d in (2, 3) for s in SIZES[d]])
def test_default_shape_gives_the_bits_of_an_explicit_one(dim, size, precision):
    nx, ny, nz = size
    sugar = (nx + ny) % 2 == 0
    cfg = lbw.RunConfig(lattice=9 if dim == 2 else 19, precision=precision, nx=nx, ny=ny, nz=nz, tau=0.6,
                        vs=2e-3, kappa_c=1e-3, gp_c=1e-4, has_s=sugar, kappa_s=1e-3 if sugar else 0.0,
                        gp_s=1e-4 if sugar else 0.0)
    fields = _fields(cfg, nx + 7 * nz)
    a = _run(cfg, fields, {})
    b = _run(cfg, fields, dict(tile_x=64, tile_y=5))
    for k in a:
        assert torch.equal(a[k], b[k]), k


# grids that take the fused 2D transport: each of its tiles, whole and ragged,
# axes shorter than its nine-cell reach, the minimal height
FUSED = [(3, 6), (7, 20), (16, 16), (33, 47), (65, 130), (200, 290), (258, 300), (512, 640)]
# one more grid per taller tile of single precision (32x24, 32x40, 32x48) and of double (32x24, 32x32)
FUSED += [(300, 560), (400, 700), (700, 1100), (480, 530)]


SCHEMES = ("weno5", "weno3", "upwind1")
# one scheme per size, all of them on two sizes
SIZE_SCHEME = [(i, s) for i in range(len(FUSED)) for j, s in enumerate(SCHEMES) if i in (1, 4) or i % 3 == j]


@pytest.mark.parametrize("precision", ["fp32_shifted", "fp64"])
@pytest.mark.parametrize("form", ["plain", "sugar", "settling", "classes"])
@pytest.mark.parametrize("periodic", [False, True])
@pytest.mark.parametrize("i,scheme", SIZE_SCHEME)
def test_fused_transport_gives_the_bits_of_the_stages(i, periodic, form, precision, scheme):
    """Several steps in one call (the fused transport, C alternating between
    two buffers, then one or two steps by stages) equal the same steps with an
    explicit tile, in every field, in the stages of the last step, through
    graph replay, and when a size class carries no S."""
    nx, ny = FUSED[i]
    extra = {}
    if form in ("sugar", "settling"):
        extra = dict(has_s=True, kappa_s=1e-3, gp_s=1e-4)
    if form == "settling":
        extra.update(vs_s=0.5, phi_c=0.1)
    if form == "classes":
        extra.update(has_s=True, kappa_s=1e-3, gp_s=1e-4, vs_s=0.3, n_classes=2, vs_class=(1e-3, 4e-3),
                     kappa_class=(1e-3, 2e-3))
    one = dict(vs=2e-3, kappa_c=1e-3) if form != "classes" else {}
    cfg = lbw.RunConfig(lattice=9, precision=precision, nx=nx, ny=ny, nz=1, tau=0.6, gp_c=1e-4, scheme_c=scheme,
                        vert_periodic=periodic, **one, **extra)
    rng = np.random.default_rng(nx + ny)
    fields = (rng.uniform(0.2, 1.0, cfg.c_shape), rng.uniform(0.0, 1.0, cfg.shape) if cfg.has_s else None,
              0.02 * rng.standard_normal((2,) + cfg.shape))
    want = _run(cfg, fields, dict(tile_x=64, tile_y=5), steps=7 + i % 2)
    got = _run(cfg, fields, {}, steps=7 + i % 2)
    for k in want:
        assert torch.equal(got[k], want[k]), k
    if i != 4:
        return
    sol = lbw.Solver(cfg, stream=torch.cuda.Stream())
    sol.set_launch(graph=1)
    sol.set_field("c", fields[0])
    if cfg.has_s:
        sol.set_field("s", fields[1])
    sol.init_equilibrium(u=fields[2])
    for n in (3, 1, 2):
        sol.step(n)
        torch.cuda.synchronize()
    sol.step(7 + i % 2 - 6)
    for k in want:
        assert torch.equal(sol.field(k), want[k]), k
    sol.close()


@pytest.mark.parametrize("precision", ["fp32_shifted", "fp64"])
def test_fused_replay_records_what_single_steps_do(precision):
    """lbw_replay on a grid with the fused transport (C passed from record to
    record) against one step at a time; records that share a C buffer fall back
    to the stages."""
    cfg = lbw.RunConfig(lattice=9, precision=precision, nx=65, ny=70, nz=1, tau=0.6, vs=2e-3, kappa_c=1e-3, gp_c=1e-4)
    c, _, u = _fields(cfg, 3)
    n = 5

    def start():
        sol = lbw.Solver(cfg)
        sol.set_field("c", c)
        sol.init_equilibrium(u=u)
        return sol

    def buffers(*shape):
        return [torch.empty(shape, dtype=sol.dtype, device="cuda") for _ in range(n)]

    sol = start()
    want = []
    for _ in range(n):
        before = sol.field("c")
        sol.step(1)
        want.append((before, sol.field("stage1"), sol.field("stage2"), sol.field("u")))
    end = {k: sol.field(k) for k in ("f", "c", "deposit")}
    sol.close()
    for shared in (False, True):
        sol = start()
        cs, a1, a2, us, rho = (buffers(*cfg.shape), buffers(*cfg.shape), buffers(*cfg.shape),
                               buffers(2, *cfg.shape), buffers(*cfg.shape))
        if shared:
            cs = [cs[0]] * n
        sol.replay(cs, a1, a2, us, rho)
        torch.cuda.synchronize()
        for i in range(n):
            if not shared:
                assert torch.equal(cs[i], want[i][0])
            assert torch.equal(a1[i], want[i][1]) and torch.equal(a2[i], want[i][2]) and torch.equal(us[i], want[i][3])
        for k in end:
            assert torch.equal(sol.field(k), end[k]), (shared, k)
        sol.close()


@pytest.mark.parametrize("precision", ["fp32_shifted", "fp64"])
@pytest.mark.parametrize("shape,launch,classes", [((65, 70, 1), {}, 1), ((65, 70, 1), {}, 2), ((70, 41, 1), dict(tile_x=64), 1),
                                                  ((64, 16, 24), {}, 2)])
@pytest.mark.parametrize("records", ["apart", "stage1_is_next_c", "stage2_is_c"])
def test_replay_with_overlapping_records(precision, shape, launch, classes, records):
    """lbw_replay, where C records coincide with stage records too (the fused
    transport then gives way to the stages, which copy C): the records written
    last, the stages and the end state are those of single steps."""
    nx, ny, nz = shape
    extra = dict(n_classes=2, vs_class=(1e-3, 4e-3), kappa_class=(1e-3, 2e-3)) if classes == 2 else dict(vs=2e-3, kappa_c=1e-3)
    cfg = lbw.RunConfig(lattice=9 if nz == 1 else 19, precision=precision, nx=nx, ny=ny, nz=nz, tau=0.6, gp_c=1e-4, **extra)
    rng = np.random.default_rng(nx)
    c = rng.uniform(0.2, 1.0, cfg.c_shape)
    dim = 2 if nz == 1 else 3
    u = 0.02 * rng.standard_normal((dim,) + cfg.shape)
    n = 4

    def start():
        sol = lbw.Solver(cfg)
        sol.set_launch(**launch)
        sol.set_field("c", c)
        sol.init_equilibrium(u=u)
        return sol

    sol = start()
    want = []
    for _ in range(n):
        before = sol.field("c")
        sol.step(1)
        want.append((before, sol.field("stage1"), sol.field("stage2"), sol.field("u")))
    end = {k: sol.field(k) for k in ("f", "c", "deposit")}
    sol.close()
    sol = start()
    buffers = lambda *s: [torch.empty(s, dtype=sol.dtype, device="cuda") for _ in range(n)]
    cs, a1, a2, us, rho = (buffers(*cfg.c_shape), buffers(*cfg.c_shape), buffers(*cfg.c_shape), buffers(dim, *cfg.shape),
                           buffers(*cfg.shape))
    if records == "stage1_is_next_c":
        a1[:-1] = cs[1:]
    elif records == "stage2_is_c":
        a2 = cs
    sol.replay(cs, a1, a2, us, rho)
    torch.cuda.synchronize()
    for i in range(n):
        if records != "stage2_is_c":
            assert torch.equal(cs[i], want[i][0])
        if records != "stage1_is_next_c" or i == n - 1:
            assert torch.equal(a1[i], want[i][1])
        assert torch.equal(a2[i], want[i][2]) and torch.equal(us[i], want[i][3])
    for k in end:
        assert torch.equal(sol.field(k), end[k]), k
    sol.close()
