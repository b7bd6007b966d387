"""The reverse faces with a WENO regularisation far below the usual 1e-6.

Any weno_eps > 0 is accepted, and where C is flat the smoothness indicators are
weno_eps itself, so the face's reverse must not form products of them that leave
the element type's range: in double precision weno_eps^2 is representable down to
1e-154 and weno_eps^3 down to 1e-103, in single precision weno_eps^2 to 1e-19.
Two states whose gradient does not depend on how small weno_eps is, so that the
oracle gives it at a moderate one:

* flat: C constant in a uniform flow, every weight the ideal one;
* step: C piecewise constant, at rest, every weight on the flat sub-stencils
  (dJ/dVs sums the faces' weighted values).

Tolerances: a few ten operations of rounding, 1e-12 in double and 1e-5 in single,
of the largest value (of the sum of the terms' sizes for dJ/dVs)."""
import dataclasses

import numpy as np
import pytest
import torch

import oracle
from paper_2106_07694_amd import lbw
from test_gpu_adjoint import _dev, oracle_cfg

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision,eps", [("fp64", 1e-99), ("fp64", 1e-101), ("fp64", 1e-110), ("fp64", 1e-150),
                                           ("fp32_shifted", 2e-19)])
@pytest.mark.parametrize("state", ["flat", "step"])
@pytest.mark.parametrize("q", [9, 19])
@pytest.mark.parametrize("variant", [0, 1])
def test_gradient_with_a_tiny_weno_eps(precision, eps, state, q, variant):
    dim = 2 if q == 9 else 3
    size = dict(nx=19, ny=23) if dim == 2 else dict(nx=9, ny=7, nz=13)
    flat = state == "flat"
    cfg = lbw.RunConfig(lattice=q, precision=precision, vs=0.03125 if flat else 0.0, kappa_c=1e-3 if flat else 0.0,
                        vert_periodic=True, fluid_mode=lbw.FLUID_FROZEN, weno_eps=eps, **size)
    ocfg = dataclasses.replace(oracle_cfg(cfg), weno_eps=1e-6 if flat else 1e-15)
    rng = np.random.default_rng(17)
    c = np.full(ocfg.shape, 0.5)
    u = np.zeros((dim,) + ocfg.shape)
    if flat:
        u += np.array([0.0625, -0.015625, 0.125][:dim]).reshape((dim, 1, 1, 1))
    else:
        v = np.arange(cfg.ny if dim == 2 else cfg.nz) >= 6
        c += 0.5 * (v[None, :, None] if dim == 2 else v[:, None, None])
    cbar_next = rng.standard_normal(ocfg.shape).astype(np.float32).astype(np.float64)
    _, want, want_vs = oracle.adjoint_step(ocfg, None, c, None, cbar_next, 0.0, u)
    dt = torch.float32 if precision == "fp32_shifted" else torch.float64
    sol = lbw.Solver(cfg)
    sol.set_launch(variant=variant)
    sol.set_field("u", u)
    cb = torch.zeros(ocfg.shape, dtype=dt, device="cuda")
    vs = torch.zeros(1, dtype=torch.float64, device="cuda")
    stage = _dev(c, dt)                     # neither state moves: both stages are C
    sol.adjoint_step(None, _dev(c, dt), None, _dev(cbar_next, dt), 0.0, None, cb, vs, sol.adjoint_workspace(),
                     a1_n=stage, a2_n=stage.clone())
    torch.cuda.synchronize()
    sol.close()
    tol = 1e-5 if precision == "fp32_shifted" else 1e-12
    assert np.max(np.abs(cb.double().cpu().numpy() - want)) <= tol * np.max(np.abs(want))
    assert abs(vs.item() - want_vs) <= tol * np.sum(np.abs(cbar_next) * c)
