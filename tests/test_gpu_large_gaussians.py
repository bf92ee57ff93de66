"""Binning of Gaussians of many tiles: the lists bit for bit against the oracle where the superblock entries
are split over the blocks by their expected number, written by a wavefront for each Gaussian of more than
32 in a window, and by one block up to two windows: few and more Gaussians on grids of more than 128
columns, mixed with small ones, and in a run in the order of depth; both modes. And their time stays
near what writing the lists takes."""
import numpy as np
import pytest
import torch

import oracle
from gpu_util import say, upload
from paper_2604_02120_amd import api

pytestmark = pytest.mark.gpu

# width, height, then (Gaussians, lowest and highest radius, lowest and highest depth) ...
SCENES = {
    "one, everywhere": (2100, 1000, [(1, 9000, 9000, 1, 2)]),
    "few, everywhere": (2100, 1000, [(300, 3000, 9000, 1, 9)]),
    "1025, large": (2100, 1000, [(1025, 300, 900, 1, 9)]),
    "4096, large and small": (2100, 700, [(4000, 0, 20, 1, 9), (96, 2000, 4000, 1, 9)]),
    "4097, large": (2100, 700, [(4097, 0, 700, 1, 9)]),
    "one block": (2100, 1000, [(3000, 0, 40, 1, 9)]),
    "two windows": (2100, 1000, [(3500, 40, 60, 1, 9)]),
    "512 ranks a block": (700, 700, [(20000, 60, 130, 1, 9)]),
    "256 ranks a block": (700, 700, [(20000, 130, 180, 1, 9)]),
    "a run in depth": (1500, 1200, [(40000, 0, 6, 1, 9), (700, 900, 2000, 20, 21), (30000, 0, 6, 30, 31)]),
    "33 entries": (4096, 300, [(2000, 2050, 2100, 1, 9)]),
    "1024 superblocks": (4096, 4096, [(40, 3000, 9000, 1, 9), (2000, 0, 30, 1, 9)]),
}


def scene(name):
    W, H, groups = SCENES[name]
    rng = np.random.default_rng(len(name))
    n = sum(g[0] for g in groups)
    radii = np.concatenate([rng.integers(g[1], g[2] + 1, g[0]) for g in groups]).astype(np.int32)
    depths = np.concatenate([rng.uniform(g[3], g[4], g[0]) for g in groups]).astype(np.float32)
    order = rng.permutation(n)
    radii, depths = radii[order], depths[order]
    i2 = (np.maximum(radii, 3) / 3.0) ** -2.0
    return dict(width=W, height=H, means2d=(rng.uniform(0, 1, (n, 2)) * [W, H]).astype(np.float32),
                conics=np.stack([i2, 0.3 * i2, 1.2 * i2], 1).astype(np.float32),
                opacity=rng.uniform(0.003, 1.0, n).astype(np.float32),
                colors=np.zeros((n, 3), np.float32), depths=depths, radii=radii)


@pytest.mark.parametrize("mode", ["rect", "visible"])
@pytest.mark.parametrize("name", list(SCENES))
def test_lists_bitexact(gpu, name, mode):
    say(f"[large] {name} {mode}")
    s = scene(name)
    W, H = s["width"], s["height"]
    vis = dict(conics=s["conics"], opacity=s["opacity"], mode=oracle.BIN_VISIBLE) if mode == "visible" else {}
    pl_ref, rg_ref = oracle.bin_tiles(s["means2d"], s["radii"], s["depths"], W, H, **vis)
    sd = upload(s, gpu)
    vis = dict(conics=sd["conics"], opacity=sd["opacity"], mode=mode) if mode == "visible" else {}
    pl, rg = api.bin_tiles(sd["means2d"], sd["radii"], sd["depths"], W, H, **vis)
    np.testing.assert_array_equal(rg.cpu().numpy().astype(np.uint32), rg_ref)
    np.testing.assert_array_equal(pl.cpu().numpy().astype(np.uint32), pl_ref)
    # the same into a workspace and a list with room for four times the pairs (as callers with a bound)
    n, cap = len(s["radii"]), 4 * len(pl_ref) + 1
    ws = api.BinWorkspace(n, cap, W, H)
    api.bin_count(sd["means2d"], sd["radii"], W, H, ws, **vis)
    room, rg2 = torch.full((cap,), -7, dtype=torch.int32, device=gpu), torch.empty_like(rg)
    st = api.bin_fill(sd["means2d"], sd["radii"], sd["depths"], W, H, ws, room, rg2, **vis)
    assert int(st.item()) == 0 and torch.equal(rg, rg2) and torch.equal(pl, room[:len(pl_ref)])
    assert bool((room[len(pl_ref):] == -7).all())


def test_time_near_the_lists(gpu):
    """4000 Gaussians on nearly all of a 4K frame's 32400 tiles each (97 M pairs or more): at most 30 times
    as long as filling the list; by one block, and a lane for each Gaussian's entries, it took 500 times."""
    W, H, n = 3840, 2160, 4000
    g = torch.Generator(device=gpu)
    g.manual_seed(5)
    means = torch.rand((n, 2), generator=g, device=gpu) * torch.tensor([W, H], device=gpu)
    depths = torch.rand((n,), generator=g, device=gpu) + 1.0
    radii = torch.full((n,), 3000, dtype=torch.int32, device=gpu)
    pl, rg = api.bin_tiles(means, radii, depths, W, H)
    assert pl.numel() > 97_000_000
    ws = api.BinWorkspace(n, pl.numel(), W, H)

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

    def binning():
        api.bin_count(means, radii, W, H, ws)
        api.bin_fill(means, radii, depths, W, H, ws, pl, rg)

    t_bin, t_fill = best(binning), best(lambda: pl.fill_(1))
    say(f"[large] binning {t_bin:.3f} ms, filling the list {t_fill:.3f} ms")
    assert t_bin <= 30.0 * t_fill
