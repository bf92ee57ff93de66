"""The deterministic backward's rows per Gaussian: at both sides of the 64 that are ranked in registers,
in grids of more tiles than are counted at a time, and for lists that name a Gaussian several times in
a tile. Repeated runs are the same bit for bit; the atomic backward, whose FP32 sums differ in their
order alone, is within the 1e-5 (normwise) that n eps allows for sums of some hundred terms."""
import numpy as np
import pytest
import torch

from gpu_util import normwise, say
from paper_2604_02120_amd import api

pytestmark = pytest.mark.gpu

# (width, height, Gaussians, standard deviation, copies of each entry in a tile's list)
CASES = {
    "one row each": (16, 16, 50, 3.0, 1),
    "around 64 rows": (160, 160, 60, 25.0, 1),
    "every tile": (700, 530, 24, 300.0, 1),
    "several per tile": (350, 300, 5, 120.0, 7),
    "several, few rows": (40, 40, 8, 10.0, 3),
}


@pytest.mark.parametrize("prec", ["fp32", "bf16"])
@pytest.mark.parametrize("name", list(CASES))
def test_rows(gpu, prec, name):
    W, H, n, sigma, copies = CASES[name]
    say(f"[det rows] {name} {prec}")
    rng = np.random.default_rng(5)
    t = lambda a: torch.tensor(np.ascontiguousarray(a, dtype=np.float32), device=gpu)  # noqa: E731
    means = t(rng.uniform(0.0, 1.0, (n, 2)) * [W, H])
    s2 = (sigma * rng.uniform(0.5, 1.5, n)) ** -2
    conics = t(np.stack([s2, 0.2 * s2, s2], 1))
    opacity, colors = t(rng.uniform(0.02, 0.2, n)), t(rng.uniform(0.0, 1.0, (n, 3)))
    radii = torch.full((n,), int(4.5 * sigma) + 1, dtype=torch.int32, device=gpu)
    pl, rg = api.bin_tiles(means, radii, t(rng.uniform(1.0, 9.0, n)), W, H)
    pl, rg = pl.repeat_interleave(copies), rg * copies
    rec = api.pack_gaussians(means, conics, opacity, colors)
    img, T, last = api.blend_forward_packed(rec, rg, pl, W, H, prec=prec)
    g = t(rng.standard_normal((3, H, W)))
    runs = [[x.clone() for x in api.blend_backward_deterministic(rec, rg, pl, W, H, T, last, g, prec=prec)]
            for _ in range(3)]
    for r in runs[1:]:
        assert all(torch.equal(a, b) for a, b in zip(runs[0], r))
    atomic = api.blend_backward_packed(rec, rg, pl, W, H, T, last, g, prec=prec)
    for a, b in zip(runs[0], atomic):
        d = normwise(a.cpu().numpy().astype(np.float64), b.cpu().numpy().astype(np.float64))
        assert d <= 1e-5, d
