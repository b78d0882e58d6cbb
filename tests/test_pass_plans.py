"""CPU tests of the launcher's choice of passes (host code of the library, called
through its C++ symbols; no device work)."""
import ctypes
import time

import numpy as np

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
