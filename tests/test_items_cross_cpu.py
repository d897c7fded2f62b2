"""Which launch groups of one-kernel solves may run together: none with a phi that
overlaps another solve's rho; against the pairwise definition, on both sides of
the size where the check sorts."""
from __future__ import annotations

import ctypes
import random

import pytest

from paper_2405_02603_amd import _lib

FIELD = 4096


def _cross(lib, rho, phi):
    f = lib._ZN3fsp8internal11items_crossEiPKPKvPKPvm
    f.restype, f.argtypes = ctypes.c_bool, [ctypes.c_int, ctypes.c_void_p, ctypes.c_void_p, ctypes.c_size_t]
    n = len(rho)
    return f(n, (ctypes.c_void_p * n)(*rho), (ctypes.c_void_p * n)(*phi), FIELD)


@pytest.mark.parametrize("count", [2, 16, 32, 33, 200])
def test_against_every_pair(count):
    lib, rng = _lib.load(), random.Random(count)
    seen = set()
    for trial in range(60):
        slots = rng.sample(range(1, 4 * count), 2 * count)
        rho, phi = [s * FIELD for s in slots[:count]], [s * FIELD for s in slots[count:]]
        if trial % 3 == 0:  # in place
            phi = list(rho)
        if trial % 2:  # one phi on, just before or just after an edge of another solve's rho
            i, j = rng.sample(range(count), 2)
            phi[i] = rho[j] + rng.choice([0, 1, -1, FIELD - 1, 1 - FIELD, FIELD, -FIELD])
        want = any(i != j and abs(phi[i] - rho[j]) < FIELD for i in range(count) for j in range(count))
        assert _cross(lib, rho, phi) == want
        seen.add(want)
    assert seen == {True, False}
    swap = [FIELD * (i + 1) for i in range(count)]
    assert _cross(lib, swap, swap[1:] + swap[:1])
