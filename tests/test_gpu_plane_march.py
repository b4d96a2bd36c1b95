"""The 3D plane-marching kernels against the oracle, bit for bit: grids of one cell, of exactly one
block, one column, row or plane more, both boundary kinds; the default's choice on both sides of
its size rule."""
import numpy as np
import pytest

import fv_inputs as fi
import oracle as O
from gpu_helpers import assert_parity, gpu_evolve, note, solver_for

pytestmark = pytest.mark.gpu

SCHEMES = [(f, r) for f in ("hllc", "hll", "rusanov") for r in ("weno3", "muscl_minmod")]
SHAPES = [(1, 1, 1), (3, 2, 20), (16, 15, 16), (17, 16, 17), (33, 14, 33)]


@pytest.mark.parametrize("n", SHAPES)
@pytest.mark.parametrize("flux,recon", SCHEMES)
def test_planes_match_oracle(flux, recon, n):
    for bc in ("periodic", "transmissive"):
        for integ in ("ssprk3", "forward_euler"):
            p = O.Problem(dim=3, n=n, eq="euler", flux=flux, recon=recon, integrator=integ, bc=(bc,) * 3)
            U0 = fi.random_smooth_state(sum(n), n[::-1], 3, batch=2)
            R, rt, rs, re = O.evolve(p, U0, 1e3, 0.2, max_steps=3)
            s = solver_for(p)
            marching = 0
            for v in range(s.num_variants()):
                s.set_variant(v)
                if s.tile()[0][2] < 16:
                    continue
                marching += 1
                note("planes", flux, recon, n, bc, integ, s.tile()[0])
                G, gt, gs, ge, st = gpu_evolve(p, U0, 1e3, 0.2, max_steps=3, mode="advance", solver=s)
                assert np.array_equal(gs, rs) and np.array_equal(gt, rt)
                assert_parity(G, R, what=f"{flux} {recon} {n} {bc} {integ} v{v}")
            assert marching


@pytest.mark.parametrize("batch", (319, 320))
def test_choice_by_size(batch):
    """16 x 14 x 17 cells are two tiles of 16 x 15 x 16: the rule lies at 320 samples."""
    p = O.Problem(dim=3, n=(16, 14, 17), eq="euler", flux="hllc", recon="weno3", integrator="ssprk3")
    few = fi.random_smooth_state(3, (17, 14, 16), 3, batch=8)
    U0 = np.ascontiguousarray(np.tile(few, (batch // 8 + 1, 1, 1, 1, 1))[:batch])
    note("planes choice", batch)
    R, rt, rs, re = O.evolve(p, few, 1e3, 0.2, max_steps=18)
    G, gt, gs, ge, st = gpu_evolve(p, U0, 1e3, 0.2, max_steps=18, mode="advance")
    assert np.all(gs == 18) and np.array_equal(gt[:8], rt)
    assert_parity(G[:8], R, what="first samples")
    assert_parity(G[-8:], R[np.arange(batch - 8, batch) % 8], what="last samples")
