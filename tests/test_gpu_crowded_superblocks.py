"""Superblocks with many chunks of entries: the lists bit for bit against the oracle at both sides of a
group of 64 chunks, for crowded superblocks beside one another and between sparse ones, with short and
long chunks and in both modes; and the time of a crowd stays near that of the same Gaussians spread over
the frame."""
import numpy as np
import pytest
import torch

import oracle
from gpu_util import say, upload
from paper_2604_02120_amd import api

pytestmark = pytest.mark.gpu

# width, height, Gaussians, then boxes (x0, y0, x1, y1) with their share of them, radius
SCENES = {
    "64 chunks": (128, 128, 64 * 256, [(20, 20, 100, 100, 1.0)], 3),
    "65 chunks": (128, 128, 64 * 256 + 1, [(20, 20, 100, 100, 1.0)], 3),
    "128 chunks": (128, 128, 128 * 256, [(20, 20, 100, 100, 1.0)], 3),
    "129 chunks": (128, 128, 128 * 256 + 1, [(20, 20, 100, 100, 1.0)], 3),
    "long chunks": (128, 128, 300000, [(0, 0, 128, 128, 1.0)], 5),
    "neighbours": (700, 500, 400000, [(0, 0, 700, 500, 0.1), (120, 120, 260, 140, 0.7),
                                      (400, 300, 420, 310, 0.2)], 9),
    "the last superblock": (640, 640, 200000, [(600, 600, 640, 640, 0.97), (0, 0, 640, 640, 0.03)], 4),
}


def scene(name):
    W, H, n, boxes, radius = SCENES[name]
    rng = np.random.default_rng(len(name))
    part = rng.choice(len(boxes), n, p=[b[4] for b in boxes])
    b = np.array([b[:4] for b in boxes])[part]
    u = rng.uniform(0, 1, (n, 2))
    i2 = rng.uniform(0.05, 0.5, n).astype(np.float32)
    return dict(width=W, height=H, means2d=(b[:, :2] + u * (b[:, 2:] - b[:, :2])).astype(np.float32),
                conics=np.stack([i2, np.float32(0.2) * i2, i2], 1),
                opacity=rng.uniform(0.002, 1.0, n).astype(np.float32),
                colors=np.zeros((n, 3), np.float32),
                depths=rng.integers(1, 5000, n).astype(np.float32),
                radii=rng.integers(1, radius + 1, n).astype(np.int32))


@pytest.mark.parametrize("mode", ["rect", "visible"])
@pytest.mark.parametrize("name", list(SCENES))
def test_lists_bitexact(gpu, name, mode):
    say(f"[crowded] {name} {mode}")
    s = scene(name)
    W, H = s["width"], s["height"]
    vis = dict(conics=s["conics"], opacity=s["opacity"], mode=oracle.BIN_VISIBLE) if mode == "visible" else {}
    pl_ref, rg_ref = oracle.bin_tiles(s["means2d"], s["radii"], s["depths"], W, H, **vis)
    sd = upload(s, gpu)
    vis = dict(conics=sd["conics"], opacity=sd["opacity"], mode=mode) if mode == "visible" else {}
    pl, rg = api.bin_tiles(sd["means2d"], sd["radii"], sd["depths"], W, H, **vis)
    np.testing.assert_array_equal(rg.cpu().numpy().astype(np.uint32), rg_ref)
    np.testing.assert_array_equal(pl.cpu().numpy().astype(np.uint32), pl_ref)


def test_time_of_a_crowd(gpu):
    """10 M Gaussians of at most 2 x 2 tiles on 128 x 128 px of a 1080p frame, against the same spread
    over the frame: with a cost per pair of chunks in a superblock it took 2.6 times as long."""
    W, H, n = 1920, 1080, 10_000_000
    g = torch.Generator(device=gpu)
    g.manual_seed(2)
    u = torch.rand((n, 2), generator=g, device=gpu)
    depths = torch.rand((n,), generator=g, device=gpu) + 1.0
    radii = torch.full((n,), 5, dtype=torch.int32, device=gpu)

    def best(means):
        ws = api.BinWorkspace(n, 0, W, H)
        pairs = int(api.bin_count(means, radii, W, H, ws).item())
        ws = api.BinWorkspace(n, pairs, W, H)
        pl = torch.empty((pairs,), dtype=torch.int32, device=gpu)
        gx, gy = api.grid(W, H)
        rg = torch.empty((gx * gy, 2), dtype=torch.int32, device=gpu)
        times = []
        for _ in range(5):
            b, e = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            b.record()
            api.bin_count(means, radii, W, H, ws)
            api.bin_fill(means, radii, depths, W, H, ws, pl, rg)
            e.record()
            e.synchronize()
            times.append(b.elapsed_time(e))
        return min(times)

    spread = best((u * torch.tensor([W, H], device=gpu)).contiguous())
    crowd = best((u * 128.0 + 512.0).contiguous())
    say(f"[crowded] spread {spread:.3f} ms, crowd {crowd:.3f} ms")
    assert crowd <= 1.5 * spread
