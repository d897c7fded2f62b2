"""float64 launch groups with spectra of up to 32 MB stream past the caches: a solve
alone and in groups on both sides of that line keeps its bits, and is the
oracle's."""
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
