"""Every byte of a plan's twiddle tables in device memory, against tables made from
their definition: lengths that two roles share, both precisions, one after the
other in one process."""
from __future__ import annotations

import numpy as np
import pytest

from twiddle_util import tables

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [(48, 48, 48), (64, 64, 64), (24, 48, 96), (96, 24, 12), (128, 8, 384), (8, 256, 192)])
def test_tables_on_the_device(n):
    import torch

    from paper_2405_02603_amd import Plan

    for prec, real in (("f32", np.float32), ("f64", np.float64), ("f32", np.float32)):
        want, total = tables(n, real)
        plan = Plan(n=n, greens="hockney", prec=prec)
        torch.cuda.synchronize()
        assert plan.octant_offset == total
        raw = plan.ghat_buf[:total].cpu().numpy()
        covered = np.zeros(total, bool)
        for values, at in want:
            size = values.size * np.dtype(real).itemsize
            got = raw[at:at + size].view(real).reshape(values.shape)
            # each value is rounded once: half a unit in the last place of 1
            assert np.max(np.abs(got.astype(np.longdouble) - values), initial=0) <= np.finfo(real).eps / 2
            covered[at:at + size] = True
        assert not raw[~covered].any()
        plan.close()
