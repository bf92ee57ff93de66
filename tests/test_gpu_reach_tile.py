"""Only the list entries that can reach a tile are staged: with GSB_FULL_SCAN every one is. Image, final
T, last contributor and the deterministic gradients must be identical bit for bit, at list lengths
around the batches of 64, 128 and 256 entries, and for conics at the edges of the test: needles at
all angles, pixels far smaller than a pixel (coefficients beyond FP16's range), indefinite conics,
opacities at the threshold."""
import numpy as np
import pytest
import torch

import gsinputs
from gpu_util import say, upload
from paper_2604_02120_amd import _lib, api

pytestmark = pytest.mark.gpu


def scene(n, s_lo, s_hi, seed, W=48, H=33, indefinite=False, faint=False):
    rng = np.random.default_rng(seed)
    s1 = np.exp(rng.uniform(np.log(s_lo), np.log(s_hi), n))
    s2 = np.exp(rng.uniform(np.log(s_lo), np.log(s_hi), n))
    conic = gsinputs.conic_from_axes(rng.uniform(0, np.pi, n), s1, s2)
    if indefinite:
        conic[::3, 1] *= 1.5
        conic[1::3, 0] = 0.0
    opacity = rng.uniform(0.003, 0.006, n) if faint else rng.uniform(0.02, 1.0, n)
    return dict(width=W, height=H,
                means2d=(rng.uniform(-0.3, 1.3, (n, 2)) * [W, H]).astype(np.float32),
                conics=conic.astype(np.float32), opacity=opacity.astype(np.float32),
                colors=rng.uniform(0, 1, (n, 3)).astype(np.float32),
                depths=rng.uniform(1, 100, n).astype(np.float32),
                # every Gaussian is listed in every tile
                radii=np.full(n, 200, np.int32))


SCENES = {
    "1 entry": lambda: scene(1, 3.0, 9.0, 1),
    "255 entries": lambda: scene(255, 0.5, 30.0, 2),
    "256 entries": lambda: scene(256, 0.5, 30.0, 3),
    "257 entries": lambda: scene(257, 0.5, 30.0, 4),
    "all reach": lambda: scene(700, 40.0, 90.0, 5, faint=True),
    "none reach": lambda: scene(300, 0.5, 2.0, 6, W=16, H=16),
    "needles": lambda: scene(2000, 0.3, 60.0, 7),
    "subpixel": lambda: scene(2000, 0.001, 0.7, 8),
    "indefinite": lambda: scene(1500, 1.0, 20.0, 9, indefinite=True),
    "faint": lambda: scene(3000, 0.5, 40.0, 10, faint=True),
}


@pytest.mark.parametrize("prec", ["fp32", "fp16", "bf16"])
@pytest.mark.parametrize("name", list(SCENES))
def test_staging_what_reaches_changes_nothing(gpu, name, prec):
    s = SCENES[name]()
    W, H = s["width"], s["height"]
    if name == "none reach":
        s["means2d"] += np.float32(100.0)
        s["radii"] += 100
    say(f"[reach tile] {name} {prec}")
    sd = upload(s, gpu)
    pl, rg = api.bin_tiles(sd["means2d"], sd["radii"], sd["depths"], W, H)
    rec = api.pack_gaussians(sd["means2d"], sd["conics"], sd["opacity"], sd["colors"])
    gd = torch.from_numpy(gsinputs.make_dloss(W, H, 80)).to(gpu)
    bg = (0.1, 0.3, 0.2)
    outs = []
    for code in (api.prec_code(prec), api.prec_code(prec) | _lib.GSB_FULL_SCAN):
        f = api.blend_forward_packed(rec, rg, pl, W, H, bg, code)
        b = api.blend_backward_deterministic(rec, rg, pl, W, H, f[1], f[2], gd, bg, code)
        g = api.blend_backward(sd["means2d"], sd["conics"], sd["opacity"], sd["colors"], rg, pl, W,
                               H, f[1], f[2], gd, bg, code)
        outs.append(([x.cpu().numpy() for x in f], [x.cpu().numpy() for x in b],
                     [x.cpu().numpy() for x in g]))
    (f0, b0, g0), (f1, b1, g1) = outs
    for x, y in zip(f0 + b0, f1 + b1):
        np.testing.assert_array_equal(x, y)
    # the atomic sums of the two: the same terms in another order, FP32 rounding of up to ~9 tiles'
    # partial sums relative to the largest of them
    for x, y in zip(g0, g1):
        scale = max(float(np.abs(y).max()), 1e-30)
        assert float(np.abs(x - y).max()) <= 1e-5 * scale
