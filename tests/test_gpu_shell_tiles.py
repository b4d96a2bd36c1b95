"""Shell structure functions on the sides of the kernels' edges: grids one cell below, at and past
the 64-cell tile, radii 1, around the unrolling by four, and the largest of either staging width,
cube and ball, orders 1 and 2; the size rule between the two 2D kernels. Tolerance: an entry is a
sum of nonnegative terms; with n of them its relative error is below n eps / 2 for any order of
additions, and either side's pairwise stages make it far less: 1e-12 as for the other functionals."""
import numpy as np
import pytest

import fv_inputs as fi
import oracle as O
from gpu_helpers import note, solver_for, torch_gpu

pytestmark = pytest.mark.gpu


def _check(n, batch, max_h, order, ball, kinds=("euler",)):
    torch = torch_gpu()
    p = O.Problem(dim=2, n=n, eq="euler", flux="hll", recon="weno3")
    U = fi.random_smooth_state(12, (1, n[1], n[0]), 2, batch=2)
    U = np.ascontiguousarray(np.tile(U, (batch // 2, 1, 1, 1, 1)))
    note("shell tiles", n, batch, max_h, order, ball)
    S = solver_for(p).structure_shell(torch.from_numpy(U).cuda(), max_h, order, ball).cpu().numpy()
    R = O.structure_shell_batch(p, U[:2], max_h, order, ball)
    for k in (0, batch - 2):
        assert np.all(np.abs(S[k:k + 2] - R) <= 1e-12 * np.abs(R))


@pytest.mark.parametrize("order,ball", [(1, False), (2, False), (1, True), (2, True)])
@pytest.mark.parametrize("n,max_h", [((64, 64), 8), ((65, 63), 9), ((63, 129), 1), ((40, 66), 16),
                                     ((130, 40), 5), ((70, 33), 17)])
def test_tiled_shells_match_oracle(n, max_h, order, ball):
    _check(n, 32, max_h, order, ball)


@pytest.mark.parametrize("batch", (30, 32))   # 4 quantities, one tile: 120 and 128 workgroups
def test_shell_size_rule(batch):
    _check((33, 33), batch, 7, 2, False)


def test_shell_narrow_grid_keeps_small_tiles():
    _check((18, 20), 64, 6, 2, False)
