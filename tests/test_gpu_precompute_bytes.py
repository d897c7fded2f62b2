"""The device memory that fsp_precompute takes, by the stream-ordered pool's own
count, is what fsp_plan_precompute_bytes reports, on every route."""
from __future__ import annotations

import ctypes

import pytest

pytestmark = pytest.mark.gpu

USED_HIGH = 8  # hipMemPoolAttrUsedMemHigh


@pytest.mark.parametrize("n", [(8, 8, 8), (48, 96, 64), (64, 64, 64)])
@pytest.mark.parametrize("kw", [dict(greens="hockney"), dict(greens="vico_dct"), dict(greens="vico"),
                                dict(greens="hockney", grad=True), dict(greens="vico_dct", grad=True),
                                dict(greens="hockney", periodic=(0, 1, 0)), dict(greens="vico_dct", periodic=(1, 0, 0))])
def test_pool_use_is_the_reported_figure(n, kw):
    import torch

    from paper_2405_02603_amd import Plan, _lib

    plan = Plan(n=n, lo=(-1.0,) * 3, hi=(1.0,) * 3, prec="f32", **kw)
    torch.cuda.synchronize()
    hip = _lib.load()  # its own runtime's entry points
    pool, high = ctypes.c_void_p(), ctypes.c_uint64(0)
    assert hip.hipDeviceGetDefaultMemPool(ctypes.byref(pool), 0) == 0
    assert hip.hipMemPoolSetAttribute(pool, USED_HIGH, ctypes.byref(high)) == 0
    plan.precompute()
    torch.cuda.synchronize()
    assert hip.hipMemPoolGetAttribute(pool, USED_HIGH, ctypes.byref(high)) == 0
    # the pool hands out whole pages
    assert plan.precompute_bytes <= high.value <= plan.precompute_bytes + (2 << 20)
