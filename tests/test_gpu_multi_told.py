"""In a run of several grids a variant told to any of the solvers is kept: the choice by size is
made only where every solver is left to its default."""
import pytest

from gpu_helpers import note, torch_gpu
from test_gpu_choice import _march, _solver, _state

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("told", (None, 0, 1))
def test_multi_grid_keeps_a_told_variant(told):
    torch_gpu()
    from paper_1912_07645_amd.solver import evolve_multi
    ns, batches = ((64, 9), (128, 32)), (5200, 236)
    ss = [_solver(n) for n in ns]
    if told is not None:
        ss[told].set_variant(0)
    states, ts = zip(*[_state(n, b) for n, b in zip(ns, batches)])
    note("two grids, told", told)
    assert evolve_multi(ss, list(states), list(ts), 1e3, 0.2, 1) == 6   # FV_EMAXSTEPS
    assert [s.last_variant() for s in ss] == [0 if told is not None else _march(ss[0])] * 2
