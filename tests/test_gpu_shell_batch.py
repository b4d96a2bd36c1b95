"""Shell structure functions do not depend on the batch: a sample alone, in a batch below the size
rule between the two 2D kernels and in one above it gives the same bits. Grids of one tile of 64 x 64,
of several, ragged on either axis, radii around the unrolling by four and the largest of either
staging width, one at which the rule does not apply; cube and ball, orders 1 and 2."""
import numpy as np
import pytest

import fv_inputs as fi
from gpu_helpers import note, torch_gpu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("order,ball", [(1, False), (2, False), (1, True), (2, True)])
@pytest.mark.parametrize("n,max_h", [((33, 33), 7), ((64, 64), 8), ((65, 130), 9), ((70, 40), 1),
                                     ((40, 66), 16), ((129, 50), 5), ((70, 33), 17)])
def test_shells_do_not_depend_on_the_batch(n, max_h, order, ball):
    torch = torch_gpu()
    from paper_1912_07645_amd import Solver
    s = Solver(dim=2, n=n, eq="euler", flux="hll", recon="weno3", integrator="ssprk3")
    few = torch.from_numpy(fi.random_smooth_state(8, (1, n[1], n[0]), 2, batch=3)).cuda()
    note("shell batch", n, max_h, order, ball)
    alone = torch.cat([s.structure_shell(few[i:i + 1].contiguous(), max_h, order, ball) for i in range(3)])
    for batch in (3, 9, 33, 66):   # 4 quantities: 12 to 264 workgroups of one tile
        S = s.structure_shell(few.repeat(batch // 3, 1, 1, 1, 1), max_h, order, ball)
        assert torch.equal(S, alone.repeat(batch // 3, 1, 1)), batch
