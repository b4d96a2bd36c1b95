"""The tuner reads a state that work queued on the caller's stream has still to write."""
import numpy as np
import pytest

import fv_inputs as fi
from gpu_helpers import note, torch_gpu

pytestmark = pytest.mark.gpu


def test_tuner_waits_for_the_callers_stream():
    torch = torch_gpu()
    from paper_1912_07645_amd import Solver
    n, B = 256, 16
    U0 = torch.from_numpy(np.tile(fi.random_smooth_state(3, (1, n, n), 2, batch=1),
                                  (B, 1, 1, 1, 1))).cuda()
    s = Solver(dim=2, n=(n, n), eq="euler", flux="hll", recon="muscl_minmod", integrator="ssprk2")
    U = torch.zeros_like(U0)          # a density of zero is refused, if seen
    big = torch.zeros(1 << 28, dtype=torch.float64, device="cuda")
    torch.cuda.synchronize()
    note("tuner stream")
    for _ in range(10):               # some milliseconds of queued work ahead of the copy
        big.add_(1.0)
    U.copy_(U0)
    assert 0 <= s.tune(U, reps=1) < s.num_variants()
