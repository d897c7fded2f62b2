"""Whole solves in one launch (grids whose spectrum fits in LDS): every size the
kernel takes, against the oracle's direct sum, and the sizes just past its line.

Tolerances are those of every solve: 1e-12 (float64) and 1e-6 (float32) of the
norm, six times that of the RMS per element.
"""
from __future__ import annotations

import itertools

import numpy as np
import pytest

import workloads as W
from gpu_util import F32_ELEM, F32_TOL, F64_ELEM, F64_TOL, elem_err, kernel_octant, reference, rel_l2, to_dev, to_host
from oracle import direct, greens, mixed

pytestmark = pytest.mark.gpu

LO, HI = (0.0, -0.5, 0.0), (1.0, 0.75, 1.5)
LINE = {"f32": 139264, "f64": 139264}  # bytes of S


def _tiny(n, prec):
    return n[0] * 2 * n[1] * (n[2] + 1) * (8 if prec == "f32" else 16) <= LINE[prec]


@pytest.mark.parametrize("prec,tol,etol", [("f64", F64_TOL, F64_ELEM), ("f32", F32_TOL, F32_ELEM)])
@pytest.mark.parametrize("n2", [8, 12, 16, 24, 32])
def test_every_size(prec, tol, etol, n2):
    """n0, n1 up to 16 on both sides of the line, and the first sizes beyond (24 points on axis 0 or 1)."""
    import torch

    from paper_2405_02603_amd import Plan

    dtype = torch.float32 if prec == "f32" else torch.float64
    for n0, n1 in list(itertools.product((8, 12, 16), repeat=2)) + [(24, 8), (8, 24)]:
        n = (n0, n1, n2)
        rho = np.random.default_rng(n0 * 10000 + n1 * 100 + n2).standard_normal(n)
        if prec == "f32":
            rho = rho.astype(np.float32).astype(np.float64)
        ref = reference(rho, "hockney", LO, HI)
        plan = Plan(n=n, lo=LO, hi=HI, greens="hockney", prec=prec)
        plan.work_buf.fill_(255)
        r = to_dev(rho, dtype)
        got = to_host(plan.solve(r))
        assert rel_l2(got, ref) <= tol, n
        assert elem_err(got, ref) <= etol, n
        if n0 <= 16 and n1 <= 16 and _tiny(n, prec):
            assert bool((plan.work_buf == 255).all()), n  # the spectrum never left the block
        again = plan.solve(r, out=r)  # in place
        assert np.array_equal(to_host(again), got), n


@pytest.mark.parametrize("prec", ["f32", "f64"])
def test_batched_captured_periodic_and_static(prec):
    """Many items of one launch, by arguments and by a captured table, give each solo solve's bits;
    periodic axes and the static-workspace call take the same kernel."""
    import torch

    from paper_2405_02603_amd import Batch, Plan, solve_batched

    dtype = torch.float32 if prec == "f32" else torch.float64
    shapes = [(16, 16, 16), (8, 12, 24), (12, 8, 8)]
    jobs = [(n, i) for i in range(7) for n in shapes]
    plans = [Plan(n=n, lo=LO, hi=HI, greens="vico_dct", prec=prec) for n, _ in jobs]
    rhos = [torch.randn(n, device="cuda", dtype=dtype, generator=torch.Generator("cuda").manual_seed(i + 1)) for n, i in jobs]
    solo = [p.solve(r).clone() for p, r in zip(plans, rhos)]
    for a, b in zip(solo, solve_batched(plans, rhos)):
        assert torch.equal(a, b)
    batch = Batch(plans, rhos)
    for _ in range(3):
        for o in batch.outs:
            o.fill_(float("nan"))
        batch.launch()
        torch.cuda.synchronize()
        for a, b in zip(solo, batch.outs):
            assert torch.equal(a, b)
    for p, r, a in zip(plans[:3], rhos, solo):
        assert torch.equal(p.solve_static(r), a)
    tol = F32_TOL if prec == "f32" else F64_TOL
    n, periodic = (12, 16, 8), (True, False, True)
    rho = W.source_density(n, LO, HI, W.multiblob(3)).astype(np.float32 if prec == "f32" else np.float64)
    plan = Plan(n=n, lo=LO, hi=HI, greens="hockney", prec=prec, periodic=periodic)
    ref = mixed.convolve_mixed(rho.astype(np.float64), greens.hockney_octant(n, LO, HI), greens.spacing(n, LO, HI), periodic)
    assert rel_l2(to_host(plan.solve(to_dev(rho, dtype))), ref) <= tol


def test_autotuned_tiny_grid_keeps_a_right_schedule():
    """The autotuner times the one-launch solve beside the separate passes; whatever it keeps is right."""
    import torch

    from paper_2405_02603_amd import Plan, autotune_batch

    n = (16, 12, 16)
    rho = np.random.default_rng(5).standard_normal(n)
    plans = [Plan(n=n, lo=LO, hi=HI, greens="vico_dct", prec="f64") for _ in range(4)]
    r = to_dev(rho, torch.float64)
    plans[0].autotune(r)
    ref = direct.convolve(rho, kernel_octant("vico_dct", n, LO, HI), greens.spacing(n, LO, HI))
    assert rel_l2(to_host(plans[0].solve(r)), ref) <= F64_TOL
    autotune_batch(plans, [r.clone() for _ in plans], reps=2)
    for p in plans:
        assert rel_l2(to_host(p.solve(r)), ref) <= F64_TOL
