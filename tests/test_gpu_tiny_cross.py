"""Tiny grids solved together where one solve's phi is another's rho (two buffers
swapped, a ring): every solve of a launch reads its own rho before it is
overwritten, as larger grids do, through each call that runs solves together."""
from __future__ import annotations

import pytest

pytestmark = pytest.mark.gpu


def _setup(n, count, prec):
    import torch

    from paper_2405_02603_amd import Plan

    dtype = torch.float32 if prec == "f32" else torch.float64
    gen = torch.Generator("cuda").manual_seed(count)
    plans = [Plan(n=n, greens="hockney", prec=prec) for _ in range(count)]
    first = [torch.randn(n, device="cuda", dtype=dtype, generator=gen) for _ in range(count)]
    sep = Plan(n=n, greens="hockney", prec=prec)
    sep.schedule = [0] * 5
    return plans, first, [sep.solve(r).clone() for r in first]


@pytest.mark.parametrize("prec", ["f32", "f64"])
@pytest.mark.parametrize("n,count", [((16, 8, 16), 2), ((8, 16, 8), 16), ((12, 8, 24), 7)])
def test_ring_of_solves(n, count, prec):
    import torch

    from paper_2405_02603_amd import solve_batched

    plans, first, want = _setup(n, count, prec)
    for _ in range(5):
        bufs = [r.clone() for r in first]
        outs = bufs[1:] + bufs[:1]
        solve_batched(plans, bufs, outs)
        for o, w in zip(outs, want):
            assert torch.equal(o, w)


@pytest.mark.parametrize("n,count", [((16, 8, 16), 2), ((8, 12, 16), 40)])
def test_captured_ring_and_back(n, count):
    """A batch whose buffers are set to a ring, then apart, then a ring again; the graph of the
    solves apart runs one kernel each (their workspaces stay untouched)."""
    import torch

    from paper_2405_02603_amd import Batch

    plans, first, want = _setup(n, count, "f64")
    apart = [p.solve(r).clone() for p, r in zip(plans, first)]
    outs = [torch.empty_like(r) for r in first]
    batch = Batch(plans, first, outs)
    for step in range(4):
        ring = step % 2 == 1
        rhos = [r.clone() for r in first]
        phis = rhos[1:] + rhos[:1] if ring else [torch.full_like(r, float("nan")) for r in first]
        batch.set_io(rhos, phis)
        for p in plans:
            p.work_buf.fill_(255)
        batch.launch()
        torch.cuda.synchronize()
        for o, w in zip(phis, want if ring else apart):
            assert torch.equal(o, w), step
        if not ring:
            assert all(bool((p.work_buf == 255).all()) for p in plans)
    batch.close()
    bufs = [r.clone() for r in first]
    batch = Batch(plans, bufs, bufs[1:] + bufs[:1])  # a ring from the start
    batch.launch()
    torch.cuda.synchronize()
    for o, w in zip(bufs[1:] + bufs[:1], want):
        assert torch.equal(o, w)
    batch.close()


def test_in_place_solves_still_run_as_one_kernel():
    import torch

    from paper_2405_02603_amd import solve_batched

    plans, first, _ = _setup((16, 8, 16), 5, "f32")
    apart = [p.solve(r).clone() for p, r in zip(plans, first)]
    for p in plans:
        p.work_buf.fill_(255)
    bufs = [r.clone() for r in first]
    solve_batched(plans, bufs, bufs)
    torch.cuda.synchronize()
    for o, w in zip(bufs, apart):
        assert torch.equal(o, w)
    assert all(bool((p.work_buf == 255).all()) for p in plans)
