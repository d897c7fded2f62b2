"""The potential's Green's transform by axis passes, against the float64 oracle's octant.

Sizes at the edges of the kernel's shapes: fewer than four input pairs beyond a
multiple of four (n = 12), one 16-row block and a part of one (8, 24), each
wave count and row-block count (64, 128, 192, 256, 384, 512), few and many
columns, and a column count that no tile divides.

Tolerance: 1e-12 of the octant's norm and 6e-12 of its RMS per element (the
float64 bars of the solve).  Each of the three passes sums at most 513 products
of unit-roundoff terms (about sqrt(513) * 1.1e-16 = 2.5e-15), and a sample of
eq. (3) carries its argument's rounding, x = L |k| / 2 < 3000 times 1.1e-16.
"""
from __future__ import annotations

import numpy as np
import pytest

from oracle import greens, mixed

from gpu_util import F64_ELEM, F64_TOL, elem_err, rel_l2, to_host

pytestmark = pytest.mark.gpu

SIZES = [(8, 12, 24), (12, 8, 8), (48, 64, 96), (128, 24, 192), (256, 12, 16), (16, 384, 8), (8, 16, 512),
         (512, 8, 12), (64, 128, 32), (96, 96, 96)]


@pytest.mark.parametrize("n", SIZES)
@pytest.mark.parametrize("kind,periodic", [("vico_dct", (0, 0, 0)), ("hockney", (0, 0, 0)), ("hockney", (1, 0, 1)),
                                           ("hockney", (0, 1, 0))])
def test_octant_by_axes(n, kind, periodic):
    import torch

    from paper_2405_02603_amd import Plan

    lo, hi = (-0.5, 0.0, 0.25), (0.5, 1.25, 1.75)
    k = greens.hockney_octant(n, lo, hi) if kind == "hockney" else greens.vico_octant(n, lo, hi)
    if any(periodic):
        k = mixed.periodic_table(k, n, tuple(bool(p) for p in periodic))
    ref = greens.mirror_transform_octant(k) * (np.prod(greens.spacing(n, lo, hi)) / (8.0 * np.prod(n)))
    plan = Plan(n=n, lo=lo, hi=hi, greens=kind, prec="f64", periodic=periodic)
    for fill in (255, 0):  # every slot is written, whatever was there
        plan.ghat_buf.fill_(fill)
        plan.precompute()
        torch.cuda.synchronize()
        got = to_host(plan.ghat_octant())
        assert rel_l2(got, ref) <= F64_TOL
        assert elem_err(got, ref) <= F64_ELEM
    tile, tiles = plan.octant_tile, (n[2] + plan.octant_tile) // plan.octant_tile
    raw = plan.ghat_buf[plan.octant_offset:plan.octant_offset + (n[1] + 1) * tiles * (n[0] + 1) * tile * 8]
    full = raw.view(torch.float64).view(n[1] + 1, tiles, n[0] + 1, tile)
    past = full.permute(2, 0, 1, 3).reshape(n[0] + 1, n[1] + 1, tiles * tile)[:, :, n[2] + 1:]
    assert torch.count_nonzero(past) == 0  # the slots past k2 = n2 hold zeros
    single = Plan(n=n, lo=lo, hi=hi, greens=kind, prec="f32", periodic=periodic)
    assert np.array_equal(to_host(single.ghat_octant()), got.astype(np.float32).astype(np.float64))
