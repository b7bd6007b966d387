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
