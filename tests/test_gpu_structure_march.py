"""Structure functions at the edges of the marching kernels: rings of 8 to 48 lags, several
lanes to a segment, lines shorter than a staged chunk, segments of equal and of ragged length, groups
of segments that end inside a line or hold several segments of a line.

S_q(h) is a sum of squares over the cells, in an order of the kernel's own: a term is the same on
both sides, and each of the additions rounds to 2^-53 of a sum of positive terms, so the relative
difference to the oracle is below (N + 64) 2^-52 for N cells and in practice, where
roundings do not all go one way, below sqrt(N) 2^-52."""
import numpy as np
import pytest

import oracle as O
from gpu_helpers import assert_parity, note, solver_for, torch_gpu

pytestmark = pytest.mark.gpu


def _problem(n, eq):
    return O.Problem(dim=len(n), n=n, eq=eq, flux="rusanov", recon="first_order",
                     integrator="forward_euler", vel=(0.7, -0.4, 0.3))


def _s2(p, U, H):
    torch = torch_gpu()
    from paper_1912_07645_amd import Stats
    st = Stats(solver_for(p), max_h=H)
    st.accumulate(torch.from_numpy(U).cuda())
    return st.read()


@pytest.mark.parametrize("n,eq,H,B", [
    ((1031,), "advection", 41, 3),        # one line, a wavefront and more of it; 48 lags
    ((5, 7), "euler", 4, 2),              # shorter than a chunk of 8 columns; few lags
    ((33, 64), "euler", 8, 3),            # one width; whole segments along y
    ((65, 130), "euler", 25, 3),          # ragged segments; the widest ring just taken
    ((130, 66), "burgers", 64, 2),        # 2 x 32 lags, all taken
    ((64, 66), "mhd", 17, 2),             # 24 lags; fields 1..3 of 8 divided
    ((66, 34), "swe", 33, 2),             # 40 lags
    ((9, 40, 11), "euler", 8, 2),         # lines in all directions
    ((300, 270), "advection", 260, 1),    # 16 x 24 lags
])
def test_lags_and_segments(n, eq, H, B):
    p = _problem(n, eq)
    nf = {"euler": p.dim + 2, "mhd": 8, "swe": p.dim + 1}.get(eq, 1)
    U = np.random.default_rng(7).uniform(1.0, 2.0, (B, nf) + p.n[::-1])
    note("structure march", n, eq, H, B)
    out = _s2(p, U, H)
    ref = O.Stats(p, max_h=H)
    ref.accumulate(U)
    tol = (p.n[0] * p.n[1] * p.n[2] + 64) * 2.0 ** -52
    assert_parity(out["s2_mean"].cpu().numpy(), ref.s2(), tol=tol, bitwise=False, what="S2 mean")
    assert_parity(out["mean"].cpu().numpy(), ref.mean, what="mean")


def test_lags_beyond_the_rings():
    """More than 64 x 32 lags take the delayed second pass. The field repeats every 33 cells, with
    values that are multiples of 1/64 (every sum is exact), so S(h) is that of one period at h mod
    33 and zero at its multiples."""
    cell = np.random.default_rng(3).integers(64, 128, (1, 1, 1, 33, 33)) / 64.0
    ref = O.Stats(_problem((33, 33), "burgers"), max_h=32)
    ref.accumulate(cell)
    one = np.concatenate([np.zeros((1, 1)), ref.s2()], axis=1)
    H = 2100
    note("structure march", 2112, H)
    out = _s2(_problem((2112, 2112), "burgers"), np.tile(cell, (1, 1, 1, 64, 64)), H)
    want = one[:, np.arange(1, H + 1) % 33]
    assert np.all(np.abs(out["s2_mean"].cpu().numpy() - want) <= 4 * 2.0 ** -52 * want)
