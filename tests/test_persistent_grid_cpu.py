"""Persistent grids per kernel class (host only): grid_mult counts 8 workgroups
per compute unit, the unit that tuning files hold, whatever a class's own
residency; untuned grids fill the compute units."""
import ctypes

import pytest

import paper_1604_03622_amd as kstap

CLASSES = [(2, 8, 4, 0), (2, 16, 4, 0), (2, 32, 4, 0), (3, 8, 4, 0), (3, 8, 8, 0), (3, 12, 4, 0), (3, 16, 8, 0),
           (4, 16, 4, 0), (6, 8, 4, 0), (3, 8, 4, 1), (3, 16, 8, 1), (3, 16, 4, 2)]
CUS = 256


@pytest.mark.parametrize("shape", CLASSES)
def test_grid_unit_and_residency(shape):
    L = kstap.lib()
    cls = getattr(L, "_ZN5kstap12kernel_classEiiii")
    grid = getattr(L, "_ZN5kstap15persistent_gridEiii")
    cls.restype = grid.restype = ctypes.c_int
    k = cls(*shape)
    assert k >= 0
    for mult in (2, 4, 64):
        assert grid(k, CUS, mult) == 8 * CUS * mult
    twelve = shape in ((2, 8, 4, 0), (3, 8, 4, 0))   # three waves a SIMD
    assert grid(k, CUS, 1) == (12 if twelve else 8) * CUS
