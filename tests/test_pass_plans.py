"""CPU tests of the launcher's choice of passes (host code of the library, called
through its C++ symbols; no device work)."""
import ctypes
import time

import numpy as np
import pytest

from paper_2102_10340_amd import _lib


class Shape(ctypes.Structure):
    _fields_ = [("cpl", ctypes.c_int), ("rw", ctypes.c_int), ("w", ctypes.c_int),
                ("K", ctypes.c_int)]


class Plan(ctypes.Structure):
    _fields_ = [("passes", ctypes.c_longlong), ("deeper", ctypes.c_longlong), ("base", Shape),
                ("deep", Shape)]


tile_shape = _lib.lib._ZN2rd10tile_shapeEiii
tile_shape.argtypes, tile_shape.restype = [ctypes.c_int] * 3, Shape


def _us_per_call(sizes, K, calls=2000):
    best = np.inf
    for _ in range(5):
        t = time.perf_counter()
        for i in range(calls):
            tile_shape(*sizes[i % len(sizes)], K)
        best = min(best, (time.perf_counter() - t) / calls * 1e6)
    return best


def test_sizes_in_turn_cost_no_more_than_one():
    """A program that steps several grids of unlike sizes in turn does not pay for
    the choice of shapes again and again (with the tables of one size kept it paid
    18 to 34 us a call, more than a short run of a small grid takes)."""
    one = _us_per_call([(128, 128)], 10)
    for n in (2, 3, 12):
        many = _us_per_call([(128 + 32 * i, 96 + 16 * i) for i in range(n)], 10)
        assert many < one + 1.5, (n, one, many)


def test_a_new_size_is_cheap():
    """The first call for a size looks at the depth it needs only."""
    sizes = [(100 + i, 90 + 2 * i) for i in range(2000)]
    t = time.perf_counter()
    for r, c in sizes:
        tile_shape(r, c, 10)
    assert (time.perf_counter() - t) / len(sizes) * 1e6 < 8.0


tile_plan = _lib.lib._ZN2rd9tile_planEiiiixPNS_8TilePlanE
tile_plan.argtypes = [ctypes.c_int] * 4 + [ctypes.c_longlong, ctypes.c_void_p]
tile_plan.restype = ctypes.c_bool
FHN, GRAY_SCOTT, CNN = 0, 1, 2


def _plan(R, C, T, model=FHN, bc=1):
    p = Plan()
    return p if tile_plan(R, C, bc, model, T, ctypes.byref(p)) else None


@pytest.mark.parametrize("bc", [0, 1])
@pytest.mark.parametrize("R,C,T,model", [
    # few steps are bound by memory
    (777, 1301, 3, FHN), (2048, 2048, 1, FHN), (1792, 1792, 2, FHN), (2000, 600, 5, FHN),
    (1280, 1280, 4, GRAY_SCOTT), (2300, 2301, 2, CNN),
    # grids a few cells wide
    (4, 500000, 8, FHN), (2, 1000000, 50, FHN), (3000000, 1, 100, FHN), (100000, 40, 7, FHN),
    (100000, 3, 8, GRAY_SCOTT), (1, 3000000, 16, CNN),
    # grids on which the streamed passes fill the chip
    (2300, 2301, 8, FHN), (2400, 2400, 8, FHN), (2400, 2400, 20, FHN), (2300, 2298, 8, GRAY_SCOTT),
    (3100, 3333, 4, CNN), (4096, 4096, 8, CNN), (2500, 2500, 1000, FHN), (6000, 6000, 12, CNN),
    (2048, 2048, 5, FHN), (3100, 3333, 3, GRAY_SCOTT), (2400, 2400, 24, FHN), (6000, 6000, 3, CNN)])
def test_runs_the_streamed_passes_are_faster_at(R, C, T, model, bc):
    assert _plan(R, C, T, model, bc) is None


@pytest.mark.parametrize("bc", [0, 1])
@pytest.mark.parametrize("R,C,T,model", [
    (1, 1, 10, FHN), (128, 128, 10, FHN), (256, 256, 1000, FHN), (777, 1301, 300, FHN),
    (1024, 1024, 6, FHN), (10000, 33, 8, FHN), (2048, 2048, 1000, FHN), (2300, 2301, 9, FHN),
    (2048, 2048, 200, GRAY_SCOTT), (256, 256, 3, GRAY_SCOTT), (512, 512, 5, CNN),
    (2603, 2900, 39, CNN), (4096, 4096, 12, CNN),
    (1024, 1024, 5, FHN), (1000, 4000, 5, FHN), (2304, 2304, 9, FHN), (2400, 2400, 10, FHN),
    (2304, 2304, 3, GRAY_SCOTT), (2600, 2665, 7, GRAY_SCOTT), (2400, 2400, 11, GRAY_SCOTT),
    (1535, 1535, 4, CNN), (4096, 4096, 3, CNN), (4096, 4096, 9, CNN),
    (4096, 4096, 5, CNN), (3500, 3500, 7, CNN)])
def test_runs_the_resident_tiles_are_faster_at(R, C, T, model, bc):
    p = _plan(R, C, T, model, bc)
    assert p is not None
    assert p.deeper * p.deep.K + (p.passes - p.deeper) * p.base.K == T
    assert p.deeper == 0 or p.deep.K == p.base.K + 1


record_depth = _lib.lib._ZN2rd17tile_record_depthEiix
_adjoint_depth = _lib.lib._ZN2rd18tile_adjoint_depthEiixb
record_depth.argtypes = [ctypes.c_int, ctypes.c_int, ctypes.c_longlong]
_adjoint_depth.argtypes = record_depth.argtypes + [ctypes.c_bool]
record_depth.restype = _adjoint_depth.restype = ctypes.c_int


def adjoint_depth(R, C, S, chain=False):
    return _adjoint_depth(R, C, S, chain)


@pytest.mark.parametrize("R,C,S", [
    (1200, 1200, 100), (1164, 1164, 8), (1300, 1300, 16), (1480, 1480, 400), (1333, 1401, 60),
    (1023, 1025, 8), (1201, 1003, 150), (777, 1001, 10), (1500, 1002, 50), (1024, 1024, 4),
    (900, 900, 2), (500000, 1, 8), (3, 100000, 50), (600, 1000, 16), (1400, 1400, 8),
    (900, 1500, 8), (20000, 20, 100)])
def test_reverse_passes_the_streamed_pairs_are_faster_at(R, C, S):
    assert adjoint_depth(R, C, S) == 0


@pytest.mark.parametrize("R,C,S", [(1, 1, 8), (256, 256, 100), (511, 511, 8), (700, 702, 50),
                                   (1024, 1024, 8), (1024, 1024, 48), (1100, 1100, 400),
                                   (512, 512, 4), (600, 1000, 24), (900, 1500, 20),
                                   (1164, 1164, 60), (1024, 1280, 16), (701, 803, 16),
                                   (1100, 1100, 4)])
def test_reverse_passes_the_resident_tiles_are_faster_at(R, C, S):
    d = adjoint_depth(R, C, S)
    assert d >= 2 and d % 2 == 0


def test_reverse_passes_of_chained_segments():
    """Beside the next segment's recording two rounds of tiles are the faster pass."""
    for R, C in ((1400, 1400), (1300, 1300), (2048, 1000)):
        assert adjoint_depth(R, C, 8) == 0 and adjoint_depth(R, C, 8, True) == 8, (R, C)
    for R, C, S in ((1400, 1400, 16), (1333, 1401, 8), (1200, 1200, 8), (2000, 2000, 8)):
        assert adjoint_depth(R, C, S, True) == 0, (R, C)


def test_recordings_on_resident_tiles():
    for R, C, n in ((1024, 1024, 2), (900, 1500, 4), (1164, 1164, 4), (2301, 2303, 5),
                    (2, 1000000, 50), (500000, 4, 8), (2500, 2500, 50)):
        assert record_depth(R, C, n) == 0, (R, C, n)
    for R, C, n in ((256, 256, 100), (1024, 1024, 8), (1333, 1401, 20), (2301, 2303, 50)):
        assert record_depth(R, C, n) >= 6, (R, C, n)
    for R, C in ((512, 512), (900, 900), (2048, 1000), (2200, 2200)):
        assert record_depth(R, C, 4) == 4, (R, C)
