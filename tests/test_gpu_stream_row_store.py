"""float64 launch groups past 600 MB of spectra stream the axis-2 forward pass's
stores: a cache hint, so every solve keeps its bits.  One solve of each grid,
and the group without its last solves, lie below."""
from __future__ import annotations

import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,below,above", [((128, 128, 128), 8, 9), ((192, 192, 192), 2, 3), ((256, 128, 96), 5, 6)])
def test_group_equals_single_solves(n, below, above):
    import torch

    from paper_2405_02603_amd import Plan, solve_batched

    plans = [Plan(n=n, greens="hockney", prec="f64") for _ in range(above)]
    assert below * plans[0].work_bytes < 600_000_000 <= above * plans[0].work_bytes
    gen = torch.Generator("cuda").manual_seed(3)
    rhos = [torch.randn(n, device="cuda", dtype=torch.float64, generator=gen) for _ in range(above)]
    single = [p.solve(r).clone() for p, r in zip(plans, rhos)]
    for count in (below, above):
        for a, b in zip(single, solve_batched(plans[:count], rhos[:count])):
            assert torch.equal(a, b), count
