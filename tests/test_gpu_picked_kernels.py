"""A plan without a schedule runs the kernels that the library picks for its grid
(the plane pairs on n x 32 x 32, 48 x 48 and 64 x 64, one kernel where a whole
solve fits in LDS); a schedule of zeros that is set is variant 0 of each pass,
alone and in every kind of launch.

Each is told by its bits: a whole solve equals the passes run one by one, the
plane schedule or the workspace it left untouched, bit for bit.  The tolerance
against the oracle is that of every solve.  The grids are ones that no other test
tunes: a new plan of a tuned grid starts with that schedule.
"""
from __future__ import annotations

import numpy as np
import pytest

from gpu_util import F32_ELEM, F32_TOL, F64_ELEM, F64_TOL, elem_err, reference, rel_l2, to_dev, to_host

pytestmark = pytest.mark.gpu

LO, HI = (0.0, -0.5, 0.0), (1.0, 0.75, 1.5)
PLANES = [(8, 32, 32), (24, 48, 48), (12, 64, 64)]
TINY = [(12, 16, 16), (8, 12, 24)]


def _plan(n, prec, **kw):
    from paper_2405_02603_amd import Plan

    return Plan(n=n, lo=LO, hi=HI, greens="hockney", prec=prec, **kw)


def _one_by_one(plan, r):
    import torch

    out = torch.empty_like(r)
    plan.work_buf.fill_(255)
    for k in range(5):
        plan.solve_passes(r, out, k, k)
    return out


@pytest.mark.parametrize("prec,tol", [("f64", F64_TOL), ("f32", F32_TOL)])
@pytest.mark.parametrize("n", PLANES + TINY)
def test_zeros_that_are_set_are_variant_0_of_each_pass(n, prec, tol):
    import torch

    from paper_2405_02603_amd import Batch, solve_batched

    dtype = torch.float32 if prec == "f32" else torch.float64
    rng = np.random.default_rng(sum(n))
    plans = [_plan(n, prec) for _ in range(3)]
    rhos = [to_dev(rng.standard_normal(n), dtype) for _ in plans]
    want = [_one_by_one(p, r) for p, r in zip(plans, rhos)]
    for p in plans:
        p.schedule = [0] * 5
        assert p.schedule == [0] * 5
        p.work_buf.fill_(255)  # every value in the workspace a NaN
    for p, r, w in zip(plans, rhos, want):
        assert torch.equal(p.solve(r), w)
        assert not bool((p.work_buf == 255).all())  # the spectrum went through the workspace
        assert torch.equal(p.solve_static(r), w)
    for o, w in zip(solve_batched(plans, rhos), want):
        assert torch.equal(o, w)
    batch = Batch(plans, rhos)
    batch.launch()
    torch.cuda.synchronize()
    for o, w in zip(batch.outs, want):
        assert torch.equal(o, w)
    assert rel_l2(to_host(want[0]), reference(to_host(rhos[0]), "hockney", LO, HI)) <= tol


@pytest.mark.parametrize("prec,tol", [("f64", F64_TOL), ("f32", F32_TOL)])
@pytest.mark.parametrize("n,items", [((8, 32, 32), 1), ((12, 48, 48), 10), ((96, 48, 48), 6), ((128, 64, 64), 4)])
def test_a_plan_without_a_schedule_runs_the_plane_pairs(n, items, prec, tol):
    """Solves and gradients, few and many planes a launch."""
    import torch

    from paper_2405_02603_amd import _lib, solve_batched

    P = _lib.PLANE
    dtype = torch.float32 if prec == "f32" else torch.float64
    rng = np.random.default_rng(items)
    rhos = [to_dev(rng.standard_normal(n), dtype) for _ in range(items)]
    picked = [_plan(n, prec) for _ in rhos]
    planes = [_plan(n, prec) for _ in rhos]
    for p in planes:
        p.schedule = [P, P, 0, P, P]
    for a, b in zip(solve_batched(picked, rhos), solve_batched(planes, rhos)):
        assert torch.equal(a, b)
    ref = reference(to_host(rhos[-1]), "hockney", LO, HI, use_direct=False)
    assert rel_l2(to_host(picked[-1].solve(rhos[-1])), ref) <= tol
    grads = []
    for sched in (None, [P, P, 0, P, P]):
        g = _plan(n, prec, grad=True)
        if sched:
            g.schedule = sched
        grads.append([t.clone() for t in g.solve_grad(rhos[0], want_phi=True)])
    assert torch.equal(grads[0][0], grads[1][0]) and torch.equal(grads[0][1], grads[1][1])


@pytest.mark.parametrize("prec,tol,etol", [("f64", F64_TOL, F64_ELEM), ("f32", F32_TOL, F32_ELEM)])
@pytest.mark.parametrize("n12", [32, 48, 64])
@pytest.mark.parametrize("n0,items", [(8, 1), (12, 10), (64, 8), (48, 11), (96, 6)])
def test_plane_shapes_against_the_oracle(n0, items, n12, prec, tol, etol):
    """Both shapes at 48 points (the second from 513 planes a launch on), and the one at 32 and 64,
    for random data and for data that lives in the two columns that share a transform (k2 = 0 and
    k2 = n2)."""
    import torch

    from paper_2405_02603_amd import _lib, solve_batched

    P = _lib.PLANE
    dtype = torch.float32 if prec == "f32" else torch.float64
    n = (n0, n12, n12)
    rng = np.random.default_rng(n0 * 100 + n12 + 1)
    plans = [_plan(n, prec) for _ in range(items)]
    for p in plans:
        p.schedule = [P, P, 0, P, P]
    rhos = [to_dev(rng.standard_normal(n), dtype) for _ in plans]
    rhos[-1] = to_dev(1.0 + (-1.0) ** np.arange(n12) * rng.standard_normal(n[:2])[:, :, None], dtype)
    for p in plans:
        p.work_buf.fill_(255)
    outs = solve_batched(plans, rhos)
    for i in {0, items // 2, items - 1}:
        ref = reference(to_host(rhos[i]), "hockney", LO, HI)
        assert rel_l2(to_host(outs[i]), ref) <= tol, i
        assert elem_err(to_host(outs[i]), ref) <= etol, i
    r = rhos[0].clone()
    assert torch.equal(plans[0].solve(r, out=r), plans[0].solve(rhos[0]))  # in place
