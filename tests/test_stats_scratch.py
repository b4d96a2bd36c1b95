"""Device scratch of the axis structure functions, by the library's own plan (host code, no device):
never more than 1 GB unless a single sample's partial sums are, and those never more than max_h sums
per 8192 cells of every axis and quantity, beside a field's worth (what a pass with a buffer of
quantities and workgroups of 8192 cells takes), so that long lags on long lines fit the card."""
import ctypes as C
import os

import pytest

LIB = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))),
                   "paper_1912_07645_amd", "libfv.so")


def _plan():
    lib = C.CDLL(LIB)
    units = lib["_ZN3fvk8sf_unitsEiPKii"]
    units.restype = C.c_int64
    units.argtypes = [C.c_int32, C.POINTER(C.c_int32), C.c_int32]
    chunk = lib["_ZN3fvk8sf_chunkEiPKiii"]
    chunk.restype = C.c_int32
    chunk.argtypes = [C.c_int32, C.POINTER(C.c_int32), C.c_int32, C.c_int32]
    return units, chunk


GRIDS = [(1 << k,) for k in (4, 7, 10, 12, 14, 17, 20, 22, 24, 28)] + [(999983,), (8193,)]
GRIDS += [(64, 64), (256, 256), (4096, 4096), (100, 20000), (16384, 8192), (1 << 20, 40)]
GRIDS += [(40, 40, 40), (512, 512, 512), (4096, 70, 70), (2, 3, 100000)]


@pytest.mark.parametrize("n", GRIDS)
def test_scratch_stays_small(n):
    units, chunk = _plan()
    dim, nq = len(n), len(n) + 2
    n32 = (C.c_int32 * 3)(*(list(n) + [1] * (3 - dim)))
    cells = 1
    for k in n:
        cells *= k
    for max_h in sorted({1, 8, 37, 48, 49, 64, 65, 500, 1024, 1025, 2048, 4096, 4097, 9000, min(n) // 2, min(n) - 1}):
        if not 1 <= max_h < min(n):
            continue
        u, c = units(dim, n32, max_h), chunk(dim, n32, nq, max_h)
        held = 8 * nq * max_h * (u + 1)          # of one sample, with its S_q(h)
        assert 1 <= c <= 256 and (c == 1 or c * held <= 1 << 30)
        assert c == 1 or c * 8 * nq * cells <= 512 << 20
        # per axis one unit per 8192 cells, ragged ends, and the 16 units of the smallest grids
        floor = sum(-(-cells // 8192) + 1 for _ in n) + 32
        assert held <= max(1 << 30, 8 * nq * (max_h * floor + cells)), (max_h, u, floor)
