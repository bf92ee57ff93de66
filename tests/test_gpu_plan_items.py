"""A plan takes any number of (view, tile) items, also more than one launch's blocks (2^24 - 1 blocks of 256
threads), without a tuning and with either launch: 4096 views of 4160 tiles each, without Gaussians, all but the
first and the last sharing their outputs."""
import ctypes

import pytest
import torch

from gpu_util import say
from paper_2604_02120_amd import _lib, api

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("launch", [None, _lib.GSB_LAUNCH_PERSISTENT, _lib.GSB_LAUNCH_GRID])
def test_more_items_than_one_launch_holds(gpu, launch):
    W, H, n_views, bg = 1024, 1040, 4096, (0.25, 0.5, 0.75)
    gx, gy = api.grid(W, H)
    assert n_views * gx * gy > 1 << 24
    say(f"[plan items] {n_views * gx * gy} items, launch {launch}")
    ranges = torch.zeros((gx * gy, 2), dtype=torch.int32, device=gpu)
    outs = [(torch.full((3, H, W), -1.0, device=gpu), torch.full((H, W), -1.0, device=gpu),
             torch.full((H, W), -1, dtype=torch.int32, device=gpu)) for _ in range(3)]
    dL = torch.ones((3, H, W), device=gpu)
    p = ranges.data_ptr()
    views = []
    for i in range(n_views):
        image, T, last = outs[0 if i == 0 else 2 if i == n_views - 1 else 1]
        views.append(_lib.GsbView(W, H, 0, p, p, 0, 0, 0, 0, (ctypes.c_float * 3)(*bg), image.data_ptr(),
                                  T.data_ptr(), last.data_ptr(), dL.data_ptr(), 0, 0, 0, 0))
    plan = _lib.gsb_plan_create(views, _lib.GSB_FP32_PLAIN,
                               None if launch is None else _lib.GsbTuning(0, 0, 0, launch, 0))
    try:
        _lib.gsb_blend_batched_forward(plan)
        torch.cuda.synchronize()
        _lib.gsb_blend_batched_backward(plan)
        torch.cuda.synchronize()
    finally:
        _lib.gsb_plan_destroy(plan)
    for image, T, last in outs:
        for c in range(3):
            assert bool((image[c] == bg[c]).all())
        assert bool((T == 1.0).all()) and bool((last == 0).all())
