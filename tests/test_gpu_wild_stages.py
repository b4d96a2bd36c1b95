"""States that are physical at the start of a step and infinite or not a number after its first stage:
nothing stops the later stages then, so their faces read such cells beside ordinary ones, in the
marches among neighbours that were fine a row before. Every variant against the oracle: the same
cells not a number, every other value the same bits, the status FV_ENONPHYS."""
import numpy as np
import pytest

import fv_inputs as fi
import oracle as O
from gpu_helpers import note, solver_for, torch_gpu
from test_gpu_fast_faces import SHAPES

pytestmark = pytest.mark.gpu

SCHEMES = ([("euler", f, r) for f in ("rusanov", "hll", "hllc", "roe")
            for r in ("first_order", "muscl_minmod", "weno3", "eno2")] +
           [("swe", f, r) for f in ("hll", "roe", "rusanov") for r in ("first_order", "muscl_minmod", "weno3")] +
           [("mhd", f, r) for f in ("rusanov", "hll") for r in ("first_order", "muscl_minmod", "weno3")] +
           [("burgers", "hll", "weno3"), ("burgers", "rusanov", "muscl_minmod"),
            ("advection", "rusanov", "weno3"), ("advection", "hll", "muscl_minmod")])


def _state(p, seed):
    """Sample 0 ordinary; sample 1 with a few cells whose fluxes or signal speeds overflow."""
    nz, ny, nx = p.n[2], p.n[1], p.n[0]
    rng = np.random.default_rng(seed)
    if p.eq == "swe":
        U = fi.random_smooth_swe(seed, (nz, ny, nx), p.dim, batch=2)
    elif p.eq == "mhd":
        U = fi.random_smooth_mhd(seed, (nz, ny, nx), p.dim, batch=2)
    else:
        U = fi.random_smooth_state(seed, (nz, ny, nx), p.dim, batch=2)
        if p.eq != "euler":
            U = U[:, :1] - 1.0
    U = np.ascontiguousarray(U)
    cells = U[1].reshape(U.shape[1], -1)
    some = rng.choice(cells.shape[1], size=3, replace=False)
    if p.eq == "euler" or p.eq == "mhd":     # the energy flux or the jump times the speed
        E = p.dim + 1 if p.eq == "euler" else 4
        cells[0, some] = (1e10, 2.0, 1e10) if p.eq == "euler" else (1e170, 1e160, 1e165)
        cells[E, some] = (1e307, 1e300, 3e306)
    elif p.eq == "swe":                      # g h^2 / 2
        cells[0, some] = (1e200, 1e160, 1e220)
    elif p.eq == "burgers":                  # u^2 / 2
        cells[0, some] = (1e200, -1e160, 1e180)
    else:                                    # the jump
        cells[0, some] = (1.7e308, -1.7e308, 1.6e308)
        cells[0, (some + 1) % cells.shape[1]] = (-1.7e308, 1.7e308, -1.6e308)
    return U


@pytest.mark.parametrize("integ", ("ssprk2", "ssprk3"))
@pytest.mark.parametrize("dim,eq,flux,recon", [(d, *s) for d in (1, 2, 3) for s in SCHEMES
                                               if d < 3 or s[0] != "swe"])
def test_wild_stage_matches_oracle(dim, eq, flux, recon, integ):
    torch = torch_gpu()
    p = O.Problem(dim=dim, n=SHAPES[dim], eq=eq, flux=flux, recon=recon, integrator=integ,
                  vel=(0.7, -0.4, 0.3), gamma=5.0 / 3.0 if eq == "mhd" else 1.4)
    U0 = _state(p, 31 + dim)
    dt = 1e-3
    M, bad = O.max_speed(p, U0[1])
    assert not bad and np.isfinite(M)                   # physical at the start
    with np.errstate(all="ignore"):
        R = np.stack([O.step(p, u, dt) for u in U0])
    assert np.isfinite(R[0]).all() and not np.isfinite(R[1]).all()
    for v in range(solver_for(p).num_variants()):
        note("wild stage", dim, eq, flux, recon, integ, "variant", v)
        s = solver_for(p, v)
        U = torch.from_numpy(U0).cuda()
        err = torch.zeros(2, dtype=torch.int32, device="cuda")
        assert s.evolve_fixed_dt(U, dt, 1, 1e300, err) == 5
        assert s.last_variant() == v and err.tolist() == [0, 5]
        G = U.cpu().numpy()
        assert np.array_equal(G, R, equal_nan=True), f"v{v}: {np.argwhere(~((G == R) | (np.isnan(G) & np.isnan(R))))[:4].tolist()}"
