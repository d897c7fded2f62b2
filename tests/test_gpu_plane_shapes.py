"""At 48 points the plane kernels take another shape from 513 planes a launch on:
a solve alone, in a batch and in a captured batch give the same bits on both
sides, by the plane schedule and by the kernels picked without one."""
from __future__ import annotations

import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", ["f32", "f64"])
@pytest.mark.parametrize("n,items", [((96, 48, 48), 6), ((64, 48, 48), 9), ((24, 48, 48), 22)])
@pytest.mark.parametrize("schedule", [None, [4, 4, 0, 4, 4], [4, 4, 1, 4, 4]])
def test_a_solve_and_a_batch_agree(n, items, schedule, prec):
    import torch

    from paper_2405_02603_amd import Batch, Plan, solve_batched

    dtype = torch.float32 if prec == "f32" else torch.float64
    gen = torch.Generator("cuda").manual_seed(items)
    plans = [Plan(n=n, greens="hockney", prec=prec) for _ in range(items)]
    for p in plans:
        if schedule:
            p.schedule = schedule
    assert n[0] <= 512 < n[0] * items
    rhos = [torch.randn(n, device="cuda", dtype=dtype, generator=gen) for _ in plans]
    alone = [p.solve(r).clone() for p, r in zip(plans, rhos)]
    for a, b in zip(alone, solve_batched(plans, rhos)):
        assert torch.equal(a, b)
    batch = Batch(plans, rhos)
    batch.launch()
    torch.cuda.synchronize()
    for a, b in zip(alone, batch.outs):
        assert torch.equal(a, b)
    batch.close()
