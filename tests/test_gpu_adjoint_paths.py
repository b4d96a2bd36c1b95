"""The reverse stage against autograd where its tiles and its two arithmetic paths meet: grids one
cell past a tile, narrower than a halo, and states with cells whose momenta lie below the range of
the short arithmetic, on whole grids and in single cells."""
import numpy as np
import pytest

import fv_inputs as fi
import oracle as O
from oracle import adjoint_torch as AT
from gpu_helpers import note, solver_for, torch_gpu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kind", ("ordinary", "one_cell", "everywhere"))
@pytest.mark.parametrize("recon", ("first_order", "muscl_minmod"))
@pytest.mark.parametrize("nx,ny", [(17, 14), (16, 13), (33, 27), (5, 40)])
def test_reverse_stage_matches_autograd(nx, ny, recon, kind):
    torch = torch_gpu()
    from paper_1912_07645_amd.adjoint import Adjoint
    U0 = fi.random_smooth_state(8, (1, ny, nx), 2, batch=2)
    if kind == "one_cell":
        U0[0, 2, 0, ny // 2, nx // 2] *= 2.0 ** -220
    elif kind == "everywhere":
        U0[:, 2] *= 2.0 ** -220
    lamT = np.random.default_rng(5).standard_normal(U0.shape)
    # square cells of side 1/32: the oracle takes one spacing
    p = O.Problem(dim=2, n=(nx, ny), eq="euler", flux="rusanov", recon=recon, integrator="ssprk2",
                  hi=(nx / 32.0, ny / 32.0, 1.0))
    M, _ = O.max_speed(p, U0[0])
    dt = 0.2 / M
    note("reverse stage", nx, ny, recon, kind)
    adj = Adjoint(solver_for(p), 2, 3, dt, every=2)
    UT = adj.forward(torch.from_numpy(U0).cuda())
    g = adj.backward(torch.from_numpy(lamT).cuda()).cpu().numpy()
    R, _ = O.evolve_fixed_dt(p, U0, dt, 3, 1.0)
    assert np.array_equal(UT.cpu().numpy(), R)
    ref = AT.vjp_steps(U0, lamT, 32, dt, 3, recon, "ssprk2")
    assert np.linalg.norm(g - ref) <= 1e-12 * np.linalg.norm(ref)
