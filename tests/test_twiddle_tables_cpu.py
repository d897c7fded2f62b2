"""Plans share their twiddle tables: buffers of plans made from several threads at
once, the first of their sizes in the process among them, are those of plans made
one after the other."""
from __future__ import annotations

import ctypes
import itertools
import threading

from paper_2405_02603_amd import _lib

SIZES = (8, 12, 24, 48, 64)


def _create(lib, n, prec):
    d = _lib.PlanDesc()
    d.n[:] = n
    d.lo[:] = [-1.0] * 3
    d.hi[:] = [1.0] * 3
    d.greens, d.prec, d.alpha, d.g0 = 0, prec, 0.0, float("nan")
    h = ctypes.c_void_p()
    assert lib.fsp_plan_create(ctypes.byref(d), ctypes.byref(h)) == _lib.FSP_OK
    g, w, off, tile = ctypes.c_size_t(), ctypes.c_size_t(), ctypes.c_size_t(), ctypes.c_int()
    assert lib.fsp_plan_bytes(h, ctypes.byref(g), ctypes.byref(w)) == _lib.FSP_OK
    assert lib.fsp_plan_ghat_layout(h, ctypes.byref(off), ctypes.byref(tile)) == _lib.FSP_OK
    lib.fsp_plan_destroy(h)
    return g.value, w.value, off.value, tile.value


def test_plans_from_threads_have_equal_layouts():
    lib = _lib.load()
    jobs = [(n, prec) for n in itertools.product(SIZES, repeat=3) for prec in (0, 1)]
    got = [dict() for _ in range(4)]

    def work(out, step):
        for n, prec in jobs[::step]:
            out[n, prec] = _create(lib, n, prec)

    threads = [threading.Thread(target=work, args=(got[i], 1 if i % 2 else -1)) for i in range(4)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    want = {(n, prec): _create(lib, n, prec) for n, prec in jobs}
    assert all(g == want for g in got)
    # the axes' tables stay apart: each length and role its own, none mixed up by the sharing
    for (n, prec), v in want.items():
        assert v[2] % 256 == 0
        assert v[2] == sum(want[m, prec][2] for m in ((n[0], 8, 8), (8, n[1], 8), (8, 8, n[2]))) - 2 * want[(8, 8, 8), prec][2]
