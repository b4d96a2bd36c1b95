"""A tuner call that fails leaves the solver as it was: one left to its default still chooses its
kernel by size, one told a variant keeps it."""
import numpy as np
import pytest

from gpu_helpers import note, torch_gpu
from test_gpu_choice import _march, _ran, _solver, _state

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("told", (False, True))
def test_failed_tune_keeps_the_choice(told):
    from paper_1912_07645_amd import fv
    n = (52, 9)
    s = _solver(n)
    if told:
        s.set_variant(0)
    U, _ = _state(n, 4)
    U[2, 0] = -1.0                       # a density that stops the tuner's first run
    note("failed tune", told)
    with pytest.raises(fv.FVError) as e:
        s.tune(U, reps=1)
    assert e.value.status == fv.FV_ENONPHYS
    assert _ran(s, n, 6144) == (0 if told else _march(s))


def test_failed_tune_keeps_the_single_workgroup_loop():
    from paper_1912_07645_amd import Solver, fv
    s = Solver(dim=1, n=(40,), eq="euler", flux="hll", recon="muscl_minmod", integrator="ssprk2")
    small = s.num_variants() - 1
    s.set_variant(small)
    U, _ = _state((40,), 2)
    U[1, 0] = -1.0
    note("failed tune, 1D")
    with pytest.raises(fv.FVError):
        s.tune(U, reps=1)
    assert s.tile()[1] == small and _ran(s, (40,), 3) == small
