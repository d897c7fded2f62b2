"""The tuners time and keep what they name: a kept schedule gives the bits of that
schedule set on a new plan; where none is kept (one kernel picked), the workspace
stays untouched."""
from __future__ import annotations

import numpy as np
import pytest

from gpu_util import to_dev

pytestmark = pytest.mark.gpu

LO, HI = (0.0, -0.5, 0.0), (1.0, 0.75, 1.5)


@pytest.mark.parametrize("prec", ["f32", "f64"])
@pytest.mark.parametrize("n", [(32, 32, 32), (16, 12, 16)])
def test_kept_schedules(n, prec):
    import torch

    from paper_2405_02603_amd import Plan, autotune_batch

    def plan():
        return Plan(n=n, lo=LO, hi=HI, greens="hockney", prec=prec)

    dtype = torch.float32 if prec == "f32" else torch.float64
    plans = [plan() for _ in range(4)]
    r = to_dev(np.random.default_rng(2).standard_normal(n), dtype)
    assert plans[0].autotune(r, reps=2)["solve_separate"] > 0
    for together in (False, True):
        if together:
            autotune_batch(plans, [r.clone() for _ in plans], reps=2)
        for p in plans if together else plans[:1]:
            p.work_buf.fill_(255)
            got = p.solve(r)
            if bool((p.work_buf == 255).all()):
                assert n == (16, 12, 16) and p.schedule == [0] * 5
                assert torch.equal(got, p.solve_static(r))
            else:
                again = plan()
                again.schedule = p.schedule
                assert torch.equal(got, again.solve(r)), p.schedule
