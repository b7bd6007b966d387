"""Graph replay over calls that change its form (stages, one-launch transport,
streaming parity), issued back to back without a wait between them: the same bits
as the same steps launched one by one."""
import numpy as np
import pytest
import torch

from paper_2106_07694_amd import lbw

pytestmark = pytest.mark.gpu

CALLS = (2, 10, 3, 2, 1, 5, 2, 4, 10, 3, 2)


@pytest.mark.parametrize("sugar", [False, True])
@pytest.mark.parametrize("size", [(65, 130), (1200, 1000)])
def test_unsynchronised_calls_of_every_form(sugar, size):
    nx, ny = size
    extra = dict(has_s=True, kappa_s=1e-3, gp_s=1e-4) if sugar else {}
    cfg = lbw.RunConfig(lattice=9, precision="fp32_shifted", nx=nx, ny=ny, nz=1, tau=0.6, vs=2e-3, kappa_c=1e-3,
                        gp_c=1e-4, **extra)
    rng = np.random.default_rng(nx)
    c, s = rng.uniform(0.2, 1.0, cfg.shape), rng.uniform(0.0, 1.0, cfg.shape)
    u = 0.02 * rng.standard_normal((2,) + cfg.shape)
    names = ["f", "c", "u", "deposit", "stage1", "stage2"] + (["s"] if sugar else [])
    got = []
    for graph in (0, 1):
        sol = lbw.Solver(cfg, stream=torch.cuda.Stream())
        sol.set_launch(graph=graph)
        sol.set_field("c", c)
        if sugar:
            sol.set_field("s", s)
        sol.init_equilibrium(u=u)
        for _ in range(2):
            for n in CALLS:
                sol.step(n)
        got.append({k: sol.field(k) for k in names})
        sol.close()
    for k in names:
        assert torch.equal(got[0][k], got[1][k]), k
