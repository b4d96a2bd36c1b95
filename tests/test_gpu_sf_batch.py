"""Axis structure functions do not depend on the batch: few units go through a kernel of their own,
whose sums are the marching kernel's bit for bit. A batch of copies of one sample has that sample's
S_q(h) as its mean exactly (every Welford increment is zero), so one sample alone is compared with a
batch beyond the size rule: lines below, at and past a segment, ragged units, 8 to 64 lags, lags
shared by 2 to 64 lanes, more lags than a pass takes, units staged at once
and in halves, every equation's quantities; and with the oracle."""
import numpy as np
import pytest

import fv_inputs as fi
import oracle as O
from gpu_helpers import note, solver_for, torch_gpu

pytestmark = pytest.mark.gpu

CASES = [("euler", (17,), 16, 4096), ("euler", (130,), 5, 4096), ("euler", (100,), 48, 2048), ("euler", (100,), 50, 2048),
         ("euler", (700,), 600, 512), ("euler", (2300,), 2100, 128), ("euler", (9000,), 8500, 128), ("burgers", (129,), 33, 4096),
         ("euler", (256, 256), 48, 40), ("burgers", (300, 256), 41, 80), ("euler", (33, 20), 8, 1024), ("euler", (65, 130), 37, 512), ("euler", (256, 40), 24, 512),
         ("euler", (127, 129), 64, 256), ("swe", (70, 65), 40, 512), ("mhd", (40, 66), 17, 256),
         ("euler", (9, 11, 130), 7, 256), ("euler", (20, 70, 18), 16, 256), ("mhd", (30,), 20, 2048)]


@pytest.mark.parametrize("eq,n,max_h,batch", CASES)
def test_structure_functions_do_not_depend_on_the_batch(eq, n, max_h, batch):
    torch = torch_gpu()
    from paper_1912_07645_amd import Stats
    shape = (1,) * (3 - len(n)) + n[::-1]
    p = O.Problem(dim=len(n), n=n, eq=eq, flux="rusanov", recon="first_order")
    f = {"swe": fi.random_smooth_swe, "mhd": fi.random_smooth_mhd}.get(eq, fi.random_smooth_state)
    U0 = f(6, shape, len(n), batch=1)
    U0 = np.ascontiguousarray(U0[:, :1] if eq == "burgers" else U0)
    U = torch.from_numpy(U0).cuda()
    note("structure functions, batch", eq, n, max_h, batch)

    def s2(V):
        st = Stats(solver_for(p), max_h=max_h)
        st.accumulate(V)
        return st.read()["s2_mean"].cpu().numpy()

    alone = s2(U)
    for b in (2, 12, batch):   # 12: between 512 and 1024 units for 256 x 256
        assert np.array_equal(s2(U.repeat(b, 1, 1, 1, 1)), alone), b
    ref = O.Stats(p, max_h=max_h)
    ref.accumulate(U0)
    # sums of nonnegative terms: each side within n eps / 2 of the exact sum, far less in practice
    assert np.all(np.abs(alone - ref.s2()) <= 1e-12 * np.abs(ref.s2()))
