"""Small launches choose where they store (float64 spectra of up to 32 MB a launch
stream past the caches) and how many blocks the axis-0 pass takes (one or two
pencil sets a block, by rounds of resident blocks): a solve alone and in groups
on both sides of these lines keeps its bits, and is the oracle's."""
from __future__ import annotations

import numpy as np
import pytest

from gpu_util import F32_ELEM, F32_TOL, F64_ELEM, F64_TOL, elem_err, reference, rel_l2, to_dev, to_host

pytestmark = pytest.mark.gpu

LO, HI = (0.0, -0.5, 0.0), (1.0, 0.75, 1.5)


@pytest.mark.parametrize("prec,tol,etol", [("f64", F64_TOL, F64_ELEM), ("f32", F32_TOL, F32_ELEM)])
@pytest.mark.parametrize("n", [(8, 48, 96), (12, 96, 24), (16, 32, 64), (24, 64, 96), (32, 24, 64), (48, 16, 64), (64, 24, 96),
                               (96, 48, 24), (128, 24, 24), (192, 16, 12), (256, 64, 48), (384, 24, 12), (512, 12, 24)])
def test_groups_keep_a_solves_bits(n, prec, tol, etol):
    import torch

    from paper_2405_02603_amd import Plan, solve_batched

    dtype = torch.float32 if prec == "f32" else torch.float64
    rng = np.random.default_rng(sum(n))
    plans = [Plan(n=n, lo=LO, hi=HI, greens="hockney", prec=prec) for _ in range(16)]
    rhos = [to_dev(rng.standard_normal(n), dtype) for _ in plans]
    ref = reference(to_host(rhos[0]), "hockney", LO, HI)
    for schedule in (None, [0, 1, 1, 1, 0], [1, 2, 2, 2, 1]):
        for p in plans:
            if schedule:
                p.schedule = schedule
            p.work_buf.fill_(255)
        alone = [p.solve(r).clone() for p, r in zip(plans, rhos)]
        assert rel_l2(to_host(alone[0]), ref) <= tol
        assert elem_err(to_host(alone[0]), ref) <= etol
        for count in (2, 3, 5, 8, 12, 16):
            for a, b in zip(alone, solve_batched(plans[:count], rhos[:count])):
                assert torch.equal(a, b), (schedule, count)


def test_first_launch_under_capture():
    """The axis-0 pass asks the runtime for its resident blocks on its first launch, here inside a
    capture, in a process of its own."""
    import os
    import subprocess
    import sys

    code = """
import sys; sys.path.insert(0, %r)
import torch
from paper_2405_02603_amd import Batch, Plan
for prec, dtype in (("f32", torch.float32), ("f64", torch.float64)):
    plans = [Plan(n=(96, 24, 24), greens="hockney", prec=prec) for _ in range(3)]
    rhos = [torch.randn(96, 24, 24, device="cuda", dtype=dtype) for _ in plans]
    batch = Batch(plans, rhos)
    for _ in range(3):
        batch.launch()
    torch.cuda.synchronize()
    for p, r, o in zip(plans, rhos, batch.outs):
        assert torch.equal(p.solve(r), o)
print("captured")
""" % os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    run = subprocess.run([sys.executable, "-c", code], capture_output=True, text=True, timeout=100)
    assert run.returncode == 0 and "captured" in run.stdout, run.stderr[-2000:]
