"""3D plane marches over segments of even length: one plane, one segment short of, at and past the
tolerance of a quarter, remainders of one to many planes, every marching variant (about 16, 32 and 64
planes), bit for bit against the oracle."""
import numpy as np
import pytest

import fv_inputs as fi
import oracle as O
from gpu_helpers import assert_parity, gpu_evolve, note, solver_for

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("planes", (1, 15, 18, 20, 21, 25, 33, 39, 50, 81))
@pytest.mark.parametrize("flux,recon", [("hllc", "weno3"), ("hll", "muscl_minmod")])
def test_even_segments_match_oracle(flux, recon, planes):
    for bc in ("periodic", "transmissive"):
        p = O.Problem(dim=3, n=(17, 6, planes), eq="euler", flux=flux, recon=recon, integrator="ssprk2", bc=(bc,) * 3)
        U0 = fi.random_smooth_state(planes, (planes, 6, 17), 3, batch=2)
        R, rt, rs, re = O.evolve(p, U0, 1e3, 0.2, max_steps=2)
        s = solver_for(p)
        for v in range(s.num_variants()):
            s.set_variant(v)
            if s.tile()[0][2] < 16:
                continue
            note("even segments", flux, recon, planes, bc, s.tile()[0])
            G, gt, gs, ge, st = gpu_evolve(p, U0, 1e3, 0.2, max_steps=2, mode="advance", solver=s)
            assert s.last_variant() == v and np.array_equal(gs, rs) and np.array_equal(gt, rt)
            assert_parity(G, R, what=f"{flux} {recon} {planes} {bc} v{v}")
