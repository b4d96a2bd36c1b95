"""Runs of at most one chunk of steps (16), which start without a first look at the counts, against
the stop rules: nothing to do, a sample that fails at the start or on the way, step limits of one, of
the whole chunk and past it, and batches on both sides of the 1024 statuses that are read in one wait.
States, times and step counts equal the oracle's."""
import numpy as np
import pytest

import fv_inputs as fi
import oracle as O
from gpu_helpers import note, solver_for, torch_gpu

pytestmark = pytest.mark.gpu


def _run(p, U0, t0, t_end, K, fails=None, mode="advance"):
    torch = torch_gpu()
    B = U0.shape[0]
    s = solver_for(p)
    U, t = torch.from_numpy(U0).cuda(), torch.from_numpy(t0.copy()).cuda()
    n = torch.zeros(B, dtype=torch.int64, device="cuda")
    e = torch.zeros(B, dtype=torch.int32, device="cuda")
    from paper_1912_07645_amd import fv
    st = getattr(s, mode)(U, t, t_end, 0.4, K, n, e)
    if fails is None:
        assert st == 0
    else:   # the status of the first failing sample
        assert st == int(e[fails]) != 0 and f"sample {fails} failed" in fv.last_error()
    return U.cpu().numpy(), t.cpu().numpy(), n.cpu().numpy(), e.cpu().numpy()


def _problem(n):
    return O.Problem(dim=len(n), n=n, eq="euler", flux="hll", recon="muscl_minmod",
                     integrator="ssprk2")


def _state(p, B, seed=9):
    nz, ny, nx = p.n[2], p.n[1], p.n[0]
    U = fi.random_smooth_state(seed, (nz, ny, nx), p.dim, batch=3)
    return np.ascontiguousarray(np.tile(U, (-(-B // 3), 1, 1, 1, 1))[:B])


@pytest.mark.parametrize("K", (1, 5, 16, 17))
def test_nothing_to_do(K):
    p = _problem((40, 21))
    U0 = _state(p, 2)
    note("short runs idle", K)
    U, t, n, e = _run(p, U0, np.full(2, 0.5), 0.5, K)
    assert np.array_equal(U, U0) and np.all(t == 0.5) and np.all(n == 0) and np.all(e == 0)


@pytest.mark.parametrize("B", (5, 1024, 1030))
@pytest.mark.parametrize("K", (1, 4, 16, 17))
def test_a_failing_sample(K, B):
    p = _problem((33,))
    U0 = _state(p, B)
    bad = B - 2
    U0[bad, 0, 0, 0, 7] = -1.0
    note("short runs failing", K, B)
    U, t, n, e = _run(p, U0, np.zeros(B), 1e3, K, fails=bad)
    R, rt, rs, re = O.evolve(p, U0[:3], 1e3, 0.4, max_steps=K)
    for b in range(B):
        if b == bad:
            assert e[b] == 5 and n[b] == 0 and np.array_equal(U[b], U0[b])
        else:
            assert e[b] == 0 and n[b] == K and t[b] == rt[b % 3] and np.array_equal(U[b], R[b % 3])


@pytest.mark.parametrize("K", (3, 16, 17))
def test_step_limit_as_an_error_and_the_end_inside_a_chunk(K):
    p = _problem((36, 30))
    U0 = _state(p, 3)
    note("short runs limit", K)
    R, rt, rs, re = O.evolve(p, U0, 1e3, 0.4, max_steps=K)
    U, t, n, e = _run(p, U0, np.zeros(3), 1e3, K, fails=0, mode="evolve")
    assert np.all(e == 6) and np.array_equal(U, R) and np.array_equal(t, rt) and np.all(n == K)
    T = 0.6 * rt.min()
    R, rt, rs, re = O.evolve(p, U0, T, 0.4, max_steps=K)
    assert np.all(rs < K) and np.all(re == 0)
    U, t, n, e = _run(p, U0, np.zeros(3), T, K)
    assert np.array_equal(U, R) and np.all(t == T) and np.array_equal(n, rs) and np.all(e == 0)
