"""GPU parity, bit for bit, where the short face arithmetic (fv_fast.h) hands over to the general
one: cells at and beyond the ends of its exponent range, zeros among them, densities and sound
speeds outside their windows, supersonic and transonic faces, densities one rounding below a
power of two (whose reciprocals are nearly halfway cases), a cell that is not finite, and tiles
and wavefronts that hold both kinds of cells."""
import numpy as np
import pytest

import fv_inputs as fi
import oracle as O
from gpu_helpers import assert_parity, gpu_evolve, note, solver_for

pytestmark = pytest.mark.gpu

SHAPES = {1: (300,), 2: (70, 37), 3: (19, 17, 11)}
SCHEMES = ([("euler", f, r) for f in ("rusanov", "hll", "hllc", "roe")
            for r in ("first_order", "muscl_minmod", "weno3")] +
           [("swe", "hll", "muscl_minmod"), ("swe", "roe", "weno3"), ("swe", "rusanov", "weno3"),
            ("mhd", "rusanov", "muscl_minmod"), ("mhd", "hll", "weno3"),
            ("burgers", "hll", "weno3"), ("advection", "rusanov", "muscl_minmod")])
KINDS = ("low_end", "high_end", "mixed", "supersonic", "all_ones", "thin", "not_finite")


def _state(p, kind, seed):
    nz, ny, nx = p.n[2], p.n[1], p.n[0]
    rng = np.random.default_rng(seed)
    if p.eq == "euler":
        U = fi.random_smooth_state(seed, (nz, ny, nx), p.dim, batch=2)
    elif p.eq == "swe":
        U = fi.random_smooth_swe(seed, (nz, ny, nx), p.dim, batch=2)
    elif p.eq == "mhd":
        U = fi.random_smooth_mhd(seed, (nz, ny, nx), p.dim, batch=2)
    else:
        U = fi.random_smooth_state(seed, (nz, ny, nx), p.dim, batch=2)[:, :1] - 1.0
    U = np.ascontiguousarray(U)
    nf = U.shape[1]
    some = rng.random(U[:, 0].shape) < 0.02
    mom = slice(1, 1 + p.dim) if nf > 1 else slice(0, 1)
    if kind == "low_end":          # momenta at both sides of 2^-200, and zeros
        e = rng.choice([-198.0, -199.0, -200.0, -201.0, -230.0], size=U[:, mom].shape)
        U[:, mom] = np.where(rng.random(U[:, mom].shape) < 0.3, 0.0, U[:, mom] * 2.0 ** e)
    elif kind == "high_end":       # every field near 2^50 (B as the square root of the pressure)
        s = 2.0 ** rng.choice([48.0, 49.5, 51.0])
        U *= s if p.eq != "mhd" else 1.0
        if p.eq == "mhd":
            U[:, :5] *= s
            U[:, 5:] *= np.sqrt(s)
    elif kind == "mixed":          # single cells far outside among ordinary ones
        if nf > 1:
            U[:, 1][some] = 1e-300
        else:
            U[:, 0][some] = 1e-300
    elif kind == "supersonic" and nf > 1:   # either direction, and sonic faces between
        v = 4.0 * np.sin(2 * np.pi * (np.arange(nx) + 0.5) / nx)
        U[:, 1] += U[:, 0] * v
        if p.eq != "swe":
            U[:, p.dim + 1 if p.eq == "euler" else 4] += 8.0 * U[:, 0] + 8.0
    elif kind == "all_ones":       # 1 - k 2^-53: nearly uniform, reciprocals next to midpoints
        k = rng.integers(0, 4, size=U[:, 0].shape)
        U[:, 0] = 1.0 - k * 2.0 ** -53
        if nf > 1:
            U[:, 1:] = 0.0
            E = p.dim + 1 if p.eq == "euler" else (4 if p.eq == "mhd" else None)
            if E:
                U[:, E] = 2.5 + k * 2.0 ** -51
    elif kind == "thin" and p.eq == "euler":   # density and pressure below the windows in places
        U *= np.where(some[:, None], 2.0 ** -130, 1.0)
    elif kind == "not_finite":
        U[1, 0, 0, 0, nx // 2] = np.nan
    return U


@pytest.mark.parametrize("kind", KINDS)
@pytest.mark.parametrize("eq,flux,recon", SCHEMES)
@pytest.mark.parametrize("dim", (1, 2, 3))
def test_faces_match_oracle(dim, eq, flux, recon, kind):
    if eq == "swe" and dim == 3:
        pytest.skip("shallow water is 1D and 2D")
    bc = ("periodic",) * 3 if KINDS.index(kind) % 2 else ("transmissive",) * 3
    p = O.Problem(dim=dim, n=SHAPES[dim], eq=eq, flux=flux, recon=recon, integrator="ssprk2",
                  bc=bc, vel=(0.7, -0.4, 0.3), gamma=5.0 / 3.0 if eq == "mhd" else 1.4)
    U0 = _state(p, kind, 17 + dim)
    K = 2
    R, rt, rs, re = O.evolve(p, U0, 1e300, 0.2, max_steps=K)
    for v in range(solver_for(p).num_variants()):
        note("faces", dim, eq, flux, recon, kind, "variant", v)
        try:
            G, gt, gs, ge, st = gpu_evolve(p, U0, 1e300, 0.2, max_steps=K, mode="advance", variant=v)
        except Exception as e:   # a sample that left the physical states stops the call
            assert "FV_ENONPHYS" in str(e) and np.any(re == 5)
            continue
        assert np.array_equal(gs, rs) and np.array_equal(gt, rt, equal_nan=True)
        ok = np.array_equal(np.isnan(G), np.isnan(R))
        assert ok, "not-a-number cells differ"
        assert_parity(np.nan_to_num(G), np.nan_to_num(R), what=f"{dim}D {eq} {flux} {recon} {kind} v{v}")
