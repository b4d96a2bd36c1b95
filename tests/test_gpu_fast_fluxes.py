"""GPU parity, bit for bit, of the short Roe, shallow-water and ideal MHD fluxes (fv_fast.h) with the
reconstructions that the general test of the short faces leaves out, and where only they hand over:
thin layers of water, a magnetic field along the axis with the sound speed at the Alfven speed (a
discriminant of zero, and one next to it), fans around a sonic point."""
import numpy as np
import pytest

import oracle as O
from gpu_helpers import assert_parity, gpu_evolve, note, solver_for
from test_gpu_fast_faces import SHAPES, _state

pytestmark = pytest.mark.gpu

SCHEMES = [("euler", "roe", "eno2"), ("swe", "hll", "first_order"), ("swe", "roe", "muscl_minmod"),
           ("swe", "roe", "first_order"), ("swe", "rusanov", "eno2"), ("mhd", "hll", "muscl_minmod"),
           ("mhd", "rusanov", "first_order"), ("mhd", "hll", "eno2")]


def _degenerate(p, seed):
    """gamma p = B_x^2 with B along x only (and a rounding beside it in some cells)."""
    U = _state(p, "plain", seed)
    rng = np.random.default_rng(seed)
    U[:, 1:4] = 0.0
    U[:, 5:] = 0.0
    B2 = rng.choice([1.0, 4.0], size=U[:, 0].shape)
    U[:, 5] = np.sqrt(B2)
    pr = B2 / p.gamma * (1.0 + rng.integers(-1, 2, size=B2.shape) * 2.0 ** -52)
    U[:, 4] = pr / (p.gamma - 1.0) + 0.5 * B2
    return U


def _fans(p, seed):
    U = _state(p, "plain", seed)
    nx = p.n[0]
    x = (np.arange(nx) + 0.5) / nx
    c = np.sqrt(9.81 * U[:, 0]) if p.eq == "swe" else 1.2
    U[:, 1] = U[:, 0] * (c + 0.6 * np.sign(np.sin(4 * np.pi * x)))
    if p.eq == "euler":
        U[:, p.dim + 1] += 8.0
    return U


@pytest.mark.parametrize("kind", ("low_end", "mixed", "supersonic", "all_ones", "not_finite", "special"))
@pytest.mark.parametrize("eq,flux,recon", SCHEMES)
@pytest.mark.parametrize("dim", (1, 2))
def test_short_fluxes_match_oracle(dim, eq, flux, recon, kind):
    p = O.Problem(dim=dim, n=SHAPES[dim], eq=eq, flux=flux, recon=recon, integrator="ssprk2",
                  bc=("periodic",) * 3, gamma=5.0 / 3.0 if eq == "mhd" else 1.4)
    if kind != "special":
        U0 = _state(p, kind, 29 + dim)
    elif eq == "mhd":
        U0 = _degenerate(p, 5)
    else:
        U0 = _fans(p, 5)
        if eq == "swe":
            U0[1] *= 2.0 ** -104
    K = 2
    R, rt, rs, re = O.evolve(p, U0, 1e300, 0.2, max_steps=K)
    for v in range(solver_for(p).num_variants()):
        note("short fluxes", dim, eq, flux, recon, kind, "variant", v)
        try:
            G, gt, gs, ge, st = gpu_evolve(p, U0, 1e300, 0.2, max_steps=K, mode="advance", variant=v)
        except Exception as e:   # a sample that left the physical states stops the call
            assert "FV_ENONPHYS" in str(e) and np.any(re == 5)
            continue
        assert np.array_equal(gs, rs) and np.array_equal(gt, rt, equal_nan=True)
        assert np.array_equal(np.isnan(G), np.isnan(R))
        assert_parity(np.nan_to_num(G), np.nan_to_num(R), what=f"{dim}D {eq} {flux} {recon} {kind} v{v}")
