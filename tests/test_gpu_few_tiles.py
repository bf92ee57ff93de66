"""The forward of small grids, which reads each group's values ahead, against the batched launch, which
does not: the same arithmetic in the same order, so bit for bit, at both sides of the grids that take
it (512 tiles in FP32, 1024 in the GEMM forms)."""
import numpy as np
import pytest
import torch

from gpu_util import say
from paper_2604_02120_amd import api

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", ["fp32", "fp16", "bf16"])
@pytest.mark.parametrize("size", [(16, 16), (512, 256), (528, 250), (512, 512), (528, 509)])
def test_same_as_batched(gpu, prec, size):
    W, H = size
    say(f"[few tiles] {W}x{H} {prec}")
    rng = np.random.default_rng(3)
    n = max(300, W * H // 8)
    t = lambda a: torch.tensor(np.ascontiguousarray(a, dtype=np.float32), device=gpu)  # noqa: E731
    s = np.exp(rng.normal(0.7, 0.8, n))
    i2 = s ** -2
    scene = dict(width=W, height=H, means2d=t(rng.uniform(0, 1, (n, 2)) * [W, H]),
                 conics=t(np.stack([i2, 0.3 * i2, i2], 1)), opacity=t(rng.uniform(0, 1, n)),
                 colors=t(rng.uniform(0, 1, (n, 3))), depths=t(rng.uniform(1, 9, n)),
                 radii=torch.tensor(np.ceil(3.4 * s), dtype=torch.int32, device=gpu))
    plan = api.BatchedViews([scene], prec=prec, bg=(0.2, 0.1, 0.3))
    plan.bin()
    plan.forward()
    v = plan.views[0]
    a = [scene[k] for k in ("means2d", "conics", "opacity", "colors")]
    single = api.blend_forward(*a, v["ranges"], v["point_list"], W, H, (0.2, 0.1, 0.3), prec)
    packed = api.blend_forward_packed(api.pack_gaussians(*a), v["ranges"], v["point_list"], W, H,
                                      (0.2, 0.1, 0.3), prec)
    torch.cuda.synchronize()
    for k, x, y in zip(("image", "final_T", "last_contrib"), single, packed):
        assert torch.equal(x, v[k]) and torch.equal(y, v[k]), k
