"""Solves of n x 32 x 32, 48 x 48 and 64 x 64 grids by variant 0 of each pass, in
launches of as many planes as lie at the ends of the plane kernels' ranges (those
kernels: test_gpu_picked_kernels.py), against the oracle, for random data and for
data that lives in the columns k2 = 0 and k2 = n2.

Tolerances are those of every solve: 1e-12 (float64) and 1e-6 (float32) of the
norm, six times that of the RMS per element.
"""
from __future__ import annotations

import numpy as np
import pytest

from gpu_util import F32_ELEM, F32_TOL, F64_ELEM, F64_TOL, elem_err, reference, rel_l2, to_dev, to_host

pytestmark = pytest.mark.gpu

LO, HI = (0.0, -0.5, 0.0), (1.0, 0.75, 1.5)


@pytest.mark.parametrize("prec,tol,etol", [("f64", F64_TOL, F64_ELEM), ("f32", F32_TOL, F32_ELEM)])
@pytest.mark.parametrize("n12", [32, 48, 64])
@pytest.mark.parametrize("n0,items", [(8, 1), (12, 10), (16, 8), (64, 8), (48, 11)])
def test_each_shape(n0, items, n12, prec, tol, etol):
    import torch

    from paper_2405_02603_amd import Plan, solve_batched

    dtype = torch.float32 if prec == "f32" else torch.float64
    n = (n0, n12, n12)
    rng = np.random.default_rng(n0 * 100 + n12)
    plans = [Plan(n=n, lo=LO, hi=HI, greens="hockney", prec=prec) for _ in range(items)]
    for p in plans:
        p.schedule = [0] * 5
    rhos = [to_dev(rng.standard_normal(n), dtype) for _ in plans]
    rhos[-1] = to_dev(1.0 + (-1.0) ** np.arange(n12) * rng.standard_normal(n[:2])[:, :, None], dtype)
    outs = solve_batched(plans, rhos)
    for i in {0, items // 2, items - 1}:
        ref = reference(to_host(rhos[i]), "hockney", LO, HI)
        got = to_host(outs[i])
        assert rel_l2(got, ref) <= tol, i
        assert elem_err(got, ref) <= etol, i
    r = rhos[0].clone()
    assert torch.equal(plans[0].solve(r, out=r), plans[0].solve(rhos[0]))  # in place


@pytest.mark.parametrize("prec,tol", [("f64", F64_TOL), ("f32", F32_TOL)])
@pytest.mark.parametrize("n12", [32, 48, 64])
def test_passes_one_by_one(n12, prec, tol):
    """The default variants pass by pass are separate kernels, and agree with the whole solve."""
    import torch

    from paper_2405_02603_amd import Plan

    dtype = torch.float32 if prec == "f32" else torch.float64
    p = Plan(n=(24, n12, n12), greens="hockney", prec=prec)
    p.schedule = [0] * 5
    r = torch.randn(24, n12, n12, device="cuda", dtype=dtype, generator=torch.Generator("cuda").manual_seed(n12))
    whole = p.solve(r).clone()
    out = torch.full_like(r, float("nan"))
    for k in range(5):
        p.solve_passes(r, out, k, k)
    assert rel_l2(to_host(out), to_host(whole)) <= tol
