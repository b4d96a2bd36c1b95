"""A short run in which no sample takes a step (t is at t_end already) ends after its first decision:
a call limited to 16 steps costs about what one limited to 2 costs. Each of 14 further steps would add
four launches, 14 us together on this grid, to a call of about 95 us: 1.5 is between 1 and the 3 that
launching them all measures. And the state, clocks and statuses stay as they are."""
import time

import numpy as np
import pytest

import fv_inputs as fi
from gpu_helpers import note, torch_gpu

pytestmark = pytest.mark.gpu


def test_a_run_of_no_steps_does_not_depend_on_the_limit():
    torch = torch_gpu()
    from paper_1912_07645_amd import Solver
    n = 1024
    s = Solver(dim=2, n=(n, n), eq="euler", flux="hllc", recon="weno3", integrator="ssprk3")
    U = torch.from_numpy(fi.random_smooth_state(1, (1, n, n), 2, batch=1)).cuda()
    V = U.clone()
    t = torch.ones(1, dtype=torch.float64, device="cuda")
    steps = torch.full((1,), 7, dtype=torch.int64, device="cuda")
    note("empty calls")

    def call(limit):
        torch.cuda.synchronize()
        a = time.perf_counter()
        assert s.advance(U, t, 1.0, 0.4, limit, steps) == 0
        torch.cuda.synchronize()
        return time.perf_counter() - a

    times = {2: [], 16: []}
    for _ in range(40):
        for limit in times:
            times[limit].append(call(limit))
    ratio = np.median(times[16][5:]) / np.median(times[2][5:])
    assert ratio < 1.5, ratio
    assert torch.equal(U, V) and t.item() == 1.0 and steps.item() == 0
