"""Which kernel a solver left to its default runs, as fv_last_variant reports it, on both sides of the
size rules: 2D rows from three rounds of 4096 strip segments, 3D planes from 576 tiles (fewer on thin
grids), columns at least four fifths full; a told variant is kept, by every stepping call."""
import numpy as np
import pytest

import fv_inputs as fi
from gpu_helpers import note, torch_gpu

pytestmark = pytest.mark.gpu

SCHEMES = [(f, r) for f in ("hllc", "hll", "rusanov") for r in ("weno3", "muscl_minmod")]


def _solver(n, flux="hll", recon="muscl_minmod", eq="euler"):
    from paper_1912_07645_amd import Solver
    return Solver(dim=len(n), n=n, eq=eq, flux=flux, recon=recon, integrator="ssprk2")


def _march(s):
    """Index of the marching variant that the default takes: the last one with its tile."""
    from paper_1912_07645_amd import Solver
    found = None
    probe = Solver(dim=s.dim, n=s.n[:s.dim], **s.names)
    for v in range(probe.num_variants()):
        probe.set_variant(v)
        (bx, by, bz), _ = probe.tile()
        if (s.dim == 2 and bx == 64) or (s.dim == 3 and (bx, by, bz) == (16, 15, 16)):
            found = v
    return found


def _state(n, batch, eq="euler"):
    torch = torch_gpu()
    shape = tuple(list(n[::-1]) if len(n) == 3 else [1] * (3 - len(n)) + list(n[::-1]))
    f = fi.random_smooth_swe if eq == "swe" else fi.random_smooth_state
    U = torch.from_numpy(np.ascontiguousarray(f(4, shape, len(n), batch=1))).cuda()
    return U.repeat(batch, 1, 1, 1, 1), torch.zeros(batch, dtype=torch.float64, device="cuda")


def _ran(s, n, batch, eq="euler"):
    U, t = _state(n, batch, eq)
    note("choice", n, batch, s.names)
    assert s.advance(U, t, 1e3, 0.2, 1) == 0
    return s.last_variant()


@pytest.mark.parametrize("flux,recon", SCHEMES)
def test_rows_by_size(flux, recon):
    rows = 16 if recon == "weno3" else 8
    n = (52, rows + 1)                       # one strip, 13/16 full, of two segments
    s = _solver(n, flux, recon)
    assert s.last_variant() == -1
    assert _ran(s, n, 6143) == 0
    assert _ran(s, n, 6144) == _march(s) > 0
    assert _ran(_solver((51, rows + 1), flux, recon), (51, rows + 1), 6144) == 0


@pytest.mark.parametrize("flux,recon", SCHEMES)
def test_planes_by_size(flux, recon):
    n = (16, 12, 30)                         # one block of columns, four fifths full, of two tiles
    s = _solver(n, flux, recon)
    assert _ran(s, n, 287) == 0
    assert _ran(s, n, 288) == _march(s) > 0
    assert _ran(_solver((16, 11, 30), flux, recon), (16, 11, 30), 320) == 0


@pytest.mark.parametrize("n,batch,march", [((220, 30), 1600, False), ((230, 42), 1100, True)])
def test_rows_not_emptier_than_tiles(n, batch, march):
    # 256 x (30 + 4) against 5/4 of 224 x 30 cells, and 256 x (42 + 6) against 5/4 of 240 x 45
    s = _solver(n, "hllc", "weno3")
    assert _ran(s, n, batch) == (_march(s) if march else 0)


@pytest.mark.parametrize("planes,tiles", [(17, 1), (20, 1), (21, 2), (32, 2), (33, 2), (40, 3), (50, 3), (98, 7)])
def test_plane_segments_are_even(planes, tiles):
    # 16 x 15 columns: one block; a segment of up to 20 planes where that saves a short one
    n = (16, 15, planes)
    s = _solver(n, "hll", "muscl_minmod")
    whole = -(-planes // 16)
    batch = min(-(-576 // tiles), max(-(-384 // tiles), -(-640 // whole)))
    assert _ran(s, n, batch) == _march(s) > 0
    assert _ran(s, n, batch - 1) == 0


def test_no_march_where_there_is_none():
    n = (64, 9)
    s = _solver(n, "roe", "weno3")
    assert _march(s) is None and _ran(s, n, 8192) == 0


def test_told_variants_are_kept():
    torch = torch_gpu()
    from paper_1912_07645_amd import Solver
    n = (52, 9)
    s = _solver(n)
    s.set_variant(0)
    assert _ran(s, n, 6144) == 0
    s.set_variant(_march(s))
    assert _ran(s, n, 1) == _march(s)
    U, t = _state(n, 2)
    assert s.advance_noalloc(U, t, 1e3, 0.2, 1) == 0 and s.last_variant() == _march(s)
    s.set_variant(0)
    assert s.evolve_fixed_dt(U, 1e-6, 1) == 0 and s.last_variant() == 0
    one = Solver(dim=1, n=(40,), eq="euler", flux="hll", recon="muscl_minmod", integrator="ssprk2")
    one.set_variant(one.num_variants() - 1)   # the single-workgroup time loop
    assert _ran(one, (40,), 3) == one.num_variants() - 1


@pytest.mark.parametrize("batches", [(5200, 235), (5200, 236)])
def test_multi_grid_by_size(batches):
    """64 x 9 cells are two segments, 128 x 32 eight: 12288 together, or eight fewer."""
    torch = torch_gpu()
    from paper_1912_07645_amd.solver import evolve_multi
    ns = ((64, 9), (128, 32))
    ss = [_solver(n) for n in ns]
    states, ts = zip(*[_state(n, b) for n, b in zip(ns, batches)])
    note("choice, two grids", batches)
    st = evolve_multi(ss, list(states), list(ts), 1e3, 0.2, 1)
    assert st == 6   # FV_EMAXSTEPS
    want = _march(ss[0]) if 2 * batches[0] + 8 * batches[1] >= 12288 else 0
    assert [s.last_variant() for s in ss] == [want] * 2
