"""The deterministic backward of Gaussians with many rows: at both sides of what is ranked in registers
(64), counted by a block (256) and sorted by one, and on more tiles than 8 x 1024. Runs are
the same bit for bit and the gradients are within the bound that the FP32 form has for large
footprints; and its time grows with the rows: for a frame-filling Gaussian it stays near the atomic
backward's, which adds the same sums."""
import numpy as np
import pytest
import torch

import oracle
from gpu_util import PLAIN_GRAD_STRESS, normwise, say, upload
from paper_2604_02120_amd import api

pytestmark = pytest.mark.gpu


def scene(W, H, n, sigma, seed):
    rng = np.random.default_rng(seed)
    s2 = (sigma * rng.uniform(0.8, 1.2, n)) ** -2
    return dict(width=W, height=H,
                means2d=(rng.uniform(-0.1, 0.3, (n, 2)) * [W, H]).astype(np.float32),
                conics=np.stack([s2, 0.1 * s2, s2], 1).astype(np.float32),
                opacity=rng.uniform(0.02, 0.05, n).astype(np.float32),
                colors=rng.uniform(0.2, 1.0, (n, 3)).astype(np.float32),
                depths=rng.uniform(1.0, 9.0, n).astype(np.float32),
                radii=np.full(n, 3 * max(W, H), np.int32))


def det_args(s, dL, gpu, prec):
    sd = upload(s, gpu)
    W, H = s["width"], s["height"]
    pl, rg = api.bin_tiles(sd["means2d"], sd["radii"], sd["depths"], W, H)
    rec = api.pack_gaussians(sd["means2d"], sd["conics"], sd["opacity"], sd["colors"])
    _, T, last = api.blend_forward_packed(rec, rg, pl, W, H, prec=prec)
    return rec, rg, pl, W, H, T, last, torch.from_numpy(dL).to(gpu)


@pytest.mark.parametrize("prec", ["fp32", "bf16"])
# tile columns, tile rows, Gaussians: every Gaussian has a row on every tile
@pytest.mark.parametrize("tx,ty,n", [(8, 8, 5), (13, 5, 5), (17, 15, 3), (16, 16, 3), (257, 1, 3), (30, 47, 70),
                                     (100, 94, 4), (4096, 3, 2)])
def test_every_tile(gpu, prec, tx, ty, n):
    say(f"[det many rows] {tx}x{ty} tiles, {n} Gaussians, {prec}")
    W, H = 16 * tx, 16 * ty - 3
    s = scene(W, H, n, 3.0 * max(W, H), tx)
    dL = np.random.default_rng(ty).uniform(0.5, 1.5, (3, H, W)).astype(np.float32)
    a = det_args(s, dL, gpu, prec)
    assert a[2].numel() == n * tx * ty
    runs = [[x.cpu().numpy() for x in api.blend_backward_deterministic(*a, prec=prec)] for _ in range(3)]
    for r in runs[1:]:
        assert all(np.array_equal(x, y) for x, y in zip(runs[0], r))
    if prec == "fp32":
        pl, rg = oracle.bin_tiles(s["means2d"], s["radii"], s["depths"], W, H)
        ref = oracle.backward(W, H, rg, pl, s["means2d"], s["conics"], s["opacity"], s["colors"], dL)
        for k, x in zip(("dmeans2d", "dconics", "dopacity", "dcolors"), runs[0]):
            e = normwise(x.astype(np.float64), ref[k])
            assert e <= PLAIN_GRAD_STRESS, (k, e)


def test_time_grows_with_the_rows(gpu):
    """16 Gaussians on each of the 32400 tiles of a 4K frame: the backward with atomics as the measure; with
    a cost per row and per 1024 tiles the deterministic one took 33 times as long."""
    W, H = 3840, 2160
    s = scene(W, H, 16, 1500.0, 1)
    a = det_args(s, np.ones((3, H, W), np.float32), gpu, "bf16")
    ws = api.DetWorkspace(16, a[2].numel(), device=gpu)

    def best(f):
        times = []
        for _ in range(5):
            b, e = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            b.record()
            f()
            e.record()
            e.synchronize()
            times.append(b.elapsed_time(e))
        return min(times)

    atomic = best(lambda: api.blend_backward_packed(*a, prec="bf16"))
    det = best(lambda: api.blend_backward_deterministic(*a, prec="bf16", ws=ws))
    say(f"[det many rows] deterministic {det:.3f} ms, atomic {atomic:.3f} ms")
    assert det <= 4.0 * atomic
