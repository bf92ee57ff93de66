"""GSB_FULL_SCAN's forward stages every list entry in batches of 128, in two buffers in turn: image, final T
and last contributor are those of the forward that drops what cannot reach a tile, bit for bit, at list
lengths around the batches, on small grids (whose groups are read ahead) and large ones, from arrays
and records, with pixels that end early and with none that do."""
import numpy as np
import pytest
import torch

from gpu_util import say, upload
from paper_2604_02120_amd import _lib, api

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", ["fp32", "fp16", "bf16"])
@pytest.mark.parametrize("opaque", [False, True])
@pytest.mark.parametrize("n", [1, 15, 127, 128, 129, 255, 257, 385, 600])
@pytest.mark.parametrize("W,H", [(48, 33), (640, 417)])        # 9 and 1080 tiles
def test_forward(gpu, W, H, n, opaque, prec):
    say(f"[full scan] {W}x{H} n={n} opaque={opaque} {prec}")
    rng = np.random.default_rng(n)
    i2 = rng.uniform(2.0, 40.0, n) ** -2
    s = dict(width=W, height=H, means2d=(rng.uniform(-0.1, 1.1, (n, 2)) * [W, H]).astype(np.float32),
             conics=np.stack([i2, 0.3 * i2, 1.5 * i2], 1).astype(np.float32),
             opacity=(rng.uniform(0.5, 1.0, n) if opaque else rng.uniform(0.003, 0.02, n)).astype(np.float32),
             colors=rng.uniform(0.0, 1.0, (n, 3)).astype(np.float32),
             depths=rng.uniform(1.0, 9.0, n).astype(np.float32), radii=np.full(n, 2 * max(W, H), np.int32))
    sd = upload(s, gpu)
    pl, rg = api.bin_tiles(sd["means2d"], sd["radii"], sd["depths"], W, H)
    gx, gy = api.grid(W, H)
    assert pl.numel() == n * gx * gy                           # every Gaussian in every tile's list
    a = [sd[k] for k in ("means2d", "conics", "opacity", "colors")]
    rec = api.pack_gaussians(*a)
    bg, code = (0.1, 0.2, 0.3), api.prec_code(prec)
    ref = [x.cpu().numpy() for x in api.blend_forward_packed(rec, rg, pl, W, H, bg, code)]
    full = code | _lib.GSB_FULL_SCAN
    for out in (api.blend_forward_packed(rec, rg, pl, W, H, bg, full),
                api.blend_forward(*a, rg, pl, W, H, bg, full)):
        for x, y in zip(out, ref):
            np.testing.assert_array_equal(x.cpu().numpy(), y)


@pytest.mark.parametrize("prec", ["fp32", "fp16", "bf16"])
@pytest.mark.parametrize("launch", [0, 1])
@pytest.mark.parametrize("batch", [64, 128, 256])
def test_plan(gpu, batch, launch, prec):
    """The same through a plan of two views, whose lists are of 9 and of 300 entries a tile."""
    say(f"[full scan] plan batch={batch} launch={launch} {prec}")
    scenes = []
    for n, W, H in ((9, 130, 65), (300, 200, 120)):
        rng = np.random.default_rng(n)
        i2 = rng.uniform(2.0, 40.0, n) ** -2
        sd = upload(dict(width=W, height=H, means2d=(rng.uniform(-0.1, 1.1, (n, 2)) * [W, H]).astype(np.float32),
                         conics=np.stack([i2, 0.3 * i2, 1.5 * i2], 1).astype(np.float32),
                         opacity=rng.uniform(0.003, 0.5, n).astype(np.float32),
                         colors=rng.uniform(0.0, 1.0, (n, 3)).astype(np.float32),
                         depths=rng.uniform(1.0, 9.0, n).astype(np.float32),
                         radii=np.full(n, 2 * max(W, H), np.int32)), gpu)
        scenes.append(sd)
    outs = []
    for code in (api.prec_code(prec), api.prec_code(prec) | _lib.GSB_FULL_SCAN):
        bv = api.BatchedViews(scenes, prec=code, tuning=dict(batch_fwd=batch, launch=launch), bg=(0.1, 0.2, 0.3))
        bv.step()
        outs.append([v[k].cpu().numpy() for v in bv.views for k in ("image", "final_T", "last_contrib")])
        bv.close()
    for x, y in zip(*outs):
        np.testing.assert_array_equal(x, y)
