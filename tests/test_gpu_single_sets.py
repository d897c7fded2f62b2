"""The axis-0 pass with one pencil set a block (small grids) and with two (larger
launches): a solve alone takes the first, a launch of sixteen the second, and
both give the same bits; each is within the solve's tolerance of the oracle."""
from __future__ import annotations

import numpy as np
import pytest

from gpu_util import F32_ELEM, F32_TOL, F64_ELEM, F64_TOL, elem_err, reference, rel_l2, to_dev, to_host

pytestmark = pytest.mark.gpu

LO, HI = (0.0, -0.5, 0.0), (1.0, 0.75, 1.5)


@pytest.mark.parametrize("prec,tol,etol", [("f64", F64_TOL, F64_ELEM), ("f32", F32_TOL, F32_ELEM)])
@pytest.mark.parametrize("variant", [0, 1, 2])
@pytest.mark.parametrize("n", [(24, 64, 96), (64, 48, 32), (96, 96, 24), (192, 64, 48), (8, 128, 64)])
def test_one_set_and_two(n, variant, prec, tol, etol):
    import torch

    from paper_2405_02603_amd import Plan, solve_batched

    dtype = torch.float32 if prec == "f32" else torch.float64
    rng = np.random.default_rng(n[0] + variant)
    plans = [Plan(n=n, lo=LO, hi=HI, greens="hockney", prec=prec) for _ in range(16)]
    rhos = [to_dev(rng.standard_normal(n), dtype) for _ in plans]
    for p in plans:
        p.schedule = [0, 0, variant, 0, 1]
    alone = [p.solve(r).clone() for p, r in zip(plans, rhos)]
    for a, b in zip(alone, solve_batched(plans, rhos)):
        assert torch.equal(a, b)
    ref = reference(to_host(rhos[0]), "hockney", LO, HI)
    assert rel_l2(to_host(alone[0]), ref) <= tol
    assert elem_err(to_host(alone[0]), ref) <= etol
