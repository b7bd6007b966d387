"""Reversed RK stages in one kernel (tiles of 64x8 nodes in 2D, 16x4x4 in 3D)
against the face and gather kernels of launch variant 1.

Both evaluate each face with the same expressions and gather a node's products
in the same order, so every output must match bit for bit: no tolerance.  Sizes
are one below, at and one above the tile's edges, axes shorter than a stencil,
and several tiles a side."""
import numpy as np
import pytest
import torch

from paper_2106_07694_amd import lbw
from test_gpu_adjoint import _dev, _flowing, oracle_cfg

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape", [(16, 4, 8), (17, 5, 7), (15, 9, 12), (33, 3, 13), (4, 4, 41), (63, 7), (64, 8),
                                   (65, 9), (129, 25), (4, 33)])
@pytest.mark.parametrize("vper", [False, True])
@pytest.mark.parametrize("precision", ["fp64", "fp32_shifted"])
@pytest.mark.parametrize("frozen", [False, True])
def test_one_kernel_stages_equal_two_kernel_form(shape, vper, precision, frozen):
    rng = np.random.default_rng(sum(shape))
    nx, ny, nz = (*shape, 1)[:3]
    q = 9 if len(shape) == 2 else 19
    cfg = lbw.RunConfig(lattice=q, precision=precision, tau=0.7, vs=0.04, kappa_c=2e-3, gp_c=3e-3,
                        vert_periodic=vper, nx=nx, ny=ny, nz=nz,
                        fluid_mode=lbw.FLUID_FROZEN if frozen else lbw.FLUID_LBM)
    ocfg = oracle_cfg(cfg)
    f_n, c_n, u0 = _flowing(ocfg, rng)
    dt = torch.float64 if precision == "fp64" else torch.float32
    fbar_next = _dev(rng.standard_normal((q,) + ocfg.shape), dt)
    cbar_next = _dev(rng.standard_normal(ocfg.shape), dt)
    outs = []
    for variant in (0, 1):
        sol = lbw.Solver(cfg)
        sol.set_launch(variant=variant)
        if frozen:
            sol.set_field("u", u0)
        fb = torch.zeros((q,) + ocfg.shape, dtype=dt, device="cuda")
        cb = torch.zeros(ocfg.shape, dtype=dt, device="cuda")
        vs = torch.zeros(1, dtype=torch.float64, device="cuda")
        work = sol.adjoint_workspace()
        sol.adjoint_step(None if frozen else _dev(f_n, dt), _dev(c_n, dt), None if frozen else fbar_next,
                         cbar_next, 0.7, None if frozen else fb, cb, vs, work)
        torch.cuda.synchronize()
        outs.append((fb.clone(), cb.clone(), vs.clone()))
        sol.close()
    for one, two in zip(*outs):
        assert torch.equal(one, two)
