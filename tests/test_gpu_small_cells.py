"""The single-workgroup loop of first-order Rusanov schemes, whose faces combine their cells' own
terms: grids that end at, before and after the lanes of a wavefront and of the workgroup (one and two
cells per thread), both boundary kinds, one stage and three; and states outside the range of the
short reciprocal and root, in some wavefronts only. Bit for bit against the oracle."""
import numpy as np
import pytest

import fv_inputs as fi
import oracle as O
from gpu_helpers import assert_parity, gpu_evolve, note, solver_for, torch_gpu

pytestmark = pytest.mark.gpu


def _run(p, U0, what, K=6):
    R, rt, rs, rerr = O.evolve(p, U0, 1e6, 0.4, max_steps=K)
    s = solver_for(p)
    s.set_variant(s.num_variants() - 1)
    assert s.tile()[0][0] == p.n[0]
    G, gt, gs, ge, st = gpu_evolve(p, U0, 1e6, 0.4, max_steps=K, mode="advance", solver=s)
    assert np.all(rerr == 6) and np.all(ge == 0) and st == 0 and np.array_equal(gs, rs)
    assert np.array_equal(gt, rt)
    assert_parity(G, R, what=what)


@pytest.mark.parametrize("bc", ("periodic", "transmissive"))
@pytest.mark.parametrize("eq,n,integ", [
    ("euler", 2, "ssprk3"), ("euler", 63, "forward_euler"), ("euler", 64, "ssprk3"),
    ("euler", 65, "forward_euler"), ("euler", 1023, "ssprk2"), ("euler", 1024, "forward_euler"),
    ("euler", 1025, "ssprk3"), ("euler", 1278, "forward_euler"), ("swe", 64, "forward_euler"),
    ("swe", 129, "ssprk3"), ("swe", 1088, "ssprk2"), ("swe", 1918, "forward_euler")])
def test_cell_terms_at_the_lanes_ends(eq, n, integ, bc):
    torch_gpu()
    p = O.Problem(dim=1, n=(n,), eq=eq, flux="rusanov", recon="first_order", integrator=integ,
                  bc=(bc,))
    make = fi.random_smooth_swe if eq == "swe" else fi.random_smooth_state
    note("small cells", eq, n, integ, bc)
    _run(p, make(n, (1, 1, n), 1, batch=3), f"small cells {eq} {n} {integ} {bc}")


@pytest.mark.parametrize("eq", ("euler", "swe"))
def test_cells_outside_the_short_range(eq):
    """Every field scaled by 2^-130 in the second sample (the velocities stay; densities and depths
    leave [2^-100, 2^100)), and a part of the third sample's cells by 2^-102."""
    torch_gpu()
    n = 400
    p = O.Problem(dim=1, n=(n,), eq=eq, flux="rusanov", recon="first_order", integrator="ssprk2")
    make = fi.random_smooth_swe if eq == "swe" else fi.random_smooth_state
    U0 = make(5, (1, 1, n), 1, batch=3)
    U0[1] *= 2.0 ** -130
    U0[2, :, :, :, 130:150] *= 2.0 ** -102
    note("small cells range", eq)
    _run(p, U0, f"small cells range {eq}", K=3)
