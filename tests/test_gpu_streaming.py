"""Launch groups on both sides of the streaming limits give the same bits: the
limits choose cache hints, never values.  One solve of each grid lies below
them (100 and 200 MB of spectra); the batches lie between and above."""
from __future__ import annotations

import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec,count,schedule", [("f32", 3, [0] * 5), ("f32", 6, [0] * 5), ("f32", 6, [4, 4, 0, 4, 4]),
                                                 ("f32", 6, [4, 4, 2, 1, 2]), ("f64", 2, [0] * 5), ("f64", 4, [1, 2, 0, 2, 1])])
def test_batched_group_equals_single_solves(prec, count, schedule):
    import torch

    from paper_2405_02603_amd import Plan, solve_batched

    dtype = torch.float32 if prec == "f32" else torch.float64
    torch.manual_seed(7)
    rhos = [torch.randn(128, 128, 128, device="cuda", dtype=dtype) for _ in range(count)]
    plans = [Plan(n=128, greens="hockney", prec=prec) for _ in range(count)]
    for p in plans:
        p.schedule = schedule
        assert p.work_bytes < 100_000_000
    assert count * plans[0].work_bytes > 100_000_000
    single = [p.solve(r).clone() for p, r in zip(plans, rhos)]
    together = solve_batched(plans, rhos)
    torch.cuda.synchronize()
    for a, b in zip(single, together):
        assert torch.equal(a, b)
