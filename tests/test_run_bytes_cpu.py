"""A batch's groups are ordered, and its graph's branches balanced, by the bytes
of the kernels that its plans run: those picked for the grid where a plan has no
schedule, those of the schedule else."""
from __future__ import annotations

import ctypes

import pytest

from paper_2405_02603_amd import _lib

P = _lib.PLANE


@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("n,pairs,spectrum", [((32, 32, 32), 2, True), ((8, 48, 48), 2, True), ((64, 64, 64), 2, True),
                                              ((96, 96, 96), 0, True), ((32, 32, 64), 0, True),
                                              ((8, 12, 16), 0, False), ((16, 16, 16), 0, False)])
def test_bytes_of_the_kernels_that_run(n, pairs, spectrum, prec):
    lib = _lib.load()
    run = lib._ZN3fsp8internal9run_bytesEP10fsp_plan_s
    run.restype, run.argtypes = ctypes.c_double, [ctypes.c_void_p]
    d = _lib.PlanDesc()
    d.n[:], d.lo[:], d.hi[:] = list(n), [-1.0] * 3, [1.0] * 3
    d.greens, d.prec, d.alpha, d.g0, d.flags = 0, prec, 0.0, float("nan"), 0
    h = ctypes.c_void_p()
    assert lib.fsp_plan_create(ctypes.byref(d), ctypes.byref(h)) == _lib.FSP_OK
    n0, n1, n2 = n
    rb = (4, 8)[prec]
    fields = (2 * n0 * n1 * n2 + (n0 + 1) * (n1 + 1) * (n2 + 1)) * rb  # rho, phi and the octant
    rows = 2 * n0 * n1 * (n2 + 1) * rb                                 # the axis-2 spectrum
    five = fields + 12 * rows
    assert run(h) == (five - 2 * pairs * rows if spectrum else fields)
    for sched, want in (((0, 0, 0, 0, 0), five), ((1, 0, 2, 0, 1), five)) + \
            (((((P, P, 1, P, P), five - 4 * rows), ((P, P, 0, 0, 0), five - 2 * rows))) if pairs else ()):
        assert lib.fsp_plan_set_schedule(h, (ctypes.c_int * 5)(*sched)) == _lib.FSP_OK
        mb = ctypes.c_double()
        assert lib.fsp_plan_model_bytes(h, ctypes.byref(mb)) == _lib.FSP_OK
        assert run(h) == mb.value == want, sched
    lib.fsp_plan_destroy(h)
