"""Twiddle tables are made once a process for each role, length and precision and
copied into every plan: the table bytes of plans, made by several threads in a
process of their own (so that no table is there yet), against sizes computed from
the definition."""
from __future__ import annotations

import itertools
import json
import os
import subprocess
import sys

import numpy as np

from twiddle_util import radix_plans, tables

SIZES = (8, 12, 24, 48, 64, 96)
APART = (24, 64, 96)  # lengths whose six tables differ in size

CHILD = """
import ctypes, itertools, json, sys, threading
sys.path.insert(0, %r)
from paper_2405_02603_amd import _lib
lib = _lib.load()
jobs = [(n, prec) for n in itertools.product(%r, repeat=3) for prec in (0, 1)]
got = [dict() for _ in range(4)]
gate = threading.Barrier(4)

def work(out, i):
    gate.wait()
    for n, prec in (jobs if i %% 2 else jobs[::-1]):
        d = _lib.PlanDesc()
        d.n[:], d.lo[:], d.hi[:] = n, [-1.0] * 3, [1.0] * 3
        d.greens, d.prec, d.alpha, d.g0 = 0, prec, 0.0, float("nan")
        h, off = ctypes.c_void_p(), ctypes.c_size_t()
        assert lib.fsp_plan_create(ctypes.byref(d), ctypes.byref(h)) == 0
        assert lib.fsp_plan_octant_offset(h, 0, ctypes.byref(off)) == 0
        lib.fsp_plan_destroy(h)
        out["%%d %%d %%d %%d" %% (*n, prec)] = off.value

threads = [threading.Thread(target=work, args=(got[i], i)) for i in range(4)]
for t in threads: t.start()
for t in threads: t.join()
print(json.dumps(got))
"""


def test_table_bytes_from_threads_in_a_fresh_process():
    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    run = subprocess.run([sys.executable, "-c", CHILD % (root, SIZES)], capture_output=True, text=True, timeout=120)
    assert run.returncode == 0, run.stderr
    got = json.loads(run.stdout)
    for n in itertools.product(SIZES, repeat=3):
        for prec, real in ((0, np.float32), (1, np.float64)):
            want = tables(n, real)[1]
            assert [g["%d %d %d %d" % (*n, prec)] for g in got] == [want] * 4, (n, prec)


def test_sizes_tell_roles_and_precisions_apart():
    """So a table kept under another's key shows in the bytes above."""
    for m in APART:
        per = []
        for real in (np.float32, np.float64):
            edges = [t[1] for t in tables((m, m, m), real)[0][::2]] + [tables((m, m, m), real)[1]]
            per += [b - a for a, b in zip(edges, edges[1:])]
        assert len(set(per)) == 6, (m, per)
    assert [len(p) for p in radix_plans()] == [15, 15]
