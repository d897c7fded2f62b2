"""fsp_plan_precompute_bytes is what fsp_precompute allocates: on open axes the two
arrays that the axis passes go between, not the samples that they never store
(the device's own count: test_gpu_precompute_bytes.py)."""
from __future__ import annotations

import ctypes
import itertools

import pytest

from paper_2405_02603_amd import _lib

SIZES = (8, 12, 16, 24, 32, 48, 64, 96, 128, 192, 256, 384, 512)
HOCKNEY, VICO, VICO_DCT = 0, 1, 2


def _bytes(lib, n, greens, flags=0, alpha=0.0):
    d = _lib.PlanDesc()
    d.n[:], d.lo[:], d.hi[:] = list(n), [-1.0] * 3, [1.0] * 3
    d.greens, d.prec, d.alpha, d.g0, d.flags = greens, 0, alpha, float("nan"), flags
    h, out = ctypes.c_void_p(), ctypes.c_size_t()
    assert lib.fsp_plan_create(ctypes.byref(d), ctypes.byref(h)) == _lib.FSP_OK
    assert lib.fsp_plan_precompute_bytes(h, ctypes.byref(out)) == _lib.FSP_OK
    lib.fsp_plan_destroy(h)
    return out.value


def _up(v, a):
    return -(-v // a) * a


def _axis_bytes(a, b, n):
    """Arrays of a and b values and the axes' matrices: even and odd parts in blocks of 16 rows by
    4 inputs, and the row left over; one for each length."""
    images = sum(-(-m // 8) * -(-m // 32) * 128 + 4 * -(-m // 8) for m in set(n))
    return _up(8 * (_up(a, 32) + _up(b, 32) + images), 256)


def test_open_axes_store_no_samples():
    lib = _lib.load()
    for n in itertools.product(SIZES, repeat=3):
        n0, n1, n2 = n
        octant, pitch = (n0 + 1) * (n1 + 1) * (n2 + 1), _up(2 * n2 + 1, 16)
        assert _bytes(lib, n, HOCKNEY) == _axis_bytes(octant, octant, n), n
        a, b = (n0 + 1) * (2 * n1 + 1) * pitch, (n0 + 1) * (n1 + 1) * pitch
        assert _bytes(lib, n, VICO_DCT) == _axis_bytes(a, b, n), n
        # the gradient's plans keep the samples' grid for the derivative tables; the axis passes'
        # arrays fit where that grid and its first transform are
        assert a <= (2 * n0 + 1) * (2 * n1 + 1) * (2 * n2 + 1) and b <= (2 * n1 + 1) * (2 * n2 + 1) * (n0 + 1), n


@pytest.mark.parametrize("n,greens,flags", [((64, 64, 64), VICO, 0), ((64, 64, 64), VICO_DCT, 1), ((64, 64, 64), VICO_DCT, 4)])
def test_other_routes_store_the_samples(n, greens, flags):
    lib = _lib.load()
    n0, n1, n2 = n
    full = 64 * n0 * n1 * n2 if greens == VICO else (2 * n0 + 1) * (2 * n1 + 1) * (2 * n2 + 1)
    first = 16 * n1 * n2 * (n0 + 1) if greens == VICO else (n0 + 1) * (2 * n1 + 1) * (2 * n2 + 1)
    assert 8 * (full + first) < _bytes(lib, n, greens, flags) < 8 * (full + first) * 1.2
    assert _bytes(lib, n, VICO_DCT) < 0.6 * _bytes(lib, n, greens, flags)
