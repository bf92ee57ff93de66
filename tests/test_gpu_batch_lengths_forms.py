"""The backward's batches at the list lengths where their size changes, each form at its own bound: the plain
form's 1e-5 and, for the GEMM forms with BF16 among them, 1e-3. (Two tiles that list all Gaussians, none
of them opaque enough to end a pixel.)"""
import numpy as np
import pytest
import torch

import gsinputs
import oracle
from gpu_util import GEMM_GRAD, PLAIN_GRAD, normwise, say, upload, upload_bins
from paper_2604_02120_amd import api
from test_gpu_superblocks import scene

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", ["fp32", "bf16"])
@pytest.mark.parametrize("n", [1, 63, 65, 127, 129, 255, 256, 257, 511, 512, 513, 700])
def test_backward(gpu, prec, n):
    say(f"[batch lengths] n={n} {prec}")
    W, H = 32, 16
    s = scene(W, H, n, 60, 60, 7 + n)
    rng = np.random.default_rng(n)
    i2 = rng.uniform(4.0, 9.0, n).astype(np.float32) ** -2
    s["conics"] = np.stack([i2, np.float32(0.2) * i2, i2], 1)
    s["opacity"] = rng.uniform(0.005, 0.02, n).astype(np.float32)
    s["colors"] = rng.uniform(0.0, 1.0, (n, 3)).astype(np.float32)
    g = gsinputs.make_dloss(W, H, 5)
    pl_ref, rg_ref = oracle.bin_tiles(s["means2d"], s["radii"], s["depths"], W, H)
    assert len(pl_ref) == 2 * n
    ref = oracle.backward(W, H, rg_ref, pl_ref, s["means2d"], s["conics"], s["opacity"], s["colors"], g)
    sd = upload(s, gpu)
    pl, rg = upload_bins(pl_ref, rg_ref, gpu)
    a = [sd[k] for k in ("means2d", "conics", "opacity", "colors")]
    _, T, last = api.blend_forward(*a, rg, pl, W, H, prec=prec)
    gd = torch.from_numpy(g).to(gpu)
    rec = api.pack_gaussians(*a)
    outs = (api.blend_backward(*a, rg, pl, W, H, T, last, gd, prec=prec),
            api.blend_backward_packed(rec, rg, pl, W, H, T, last, gd, prec=prec),
            api.blend_backward_deterministic(rec, rg, pl, W, H, T, last, gd, prec=prec))
    for out in outs:
        for k, x in zip(("dmeans2d", "dconics", "dopacity", "dcolors"), out):
            e = normwise(x.cpu().numpy().astype(np.float64), ref[k])
            assert e <= (PLAIN_GRAD if prec == "fp32" else GEMM_GRAD), (k, e)
