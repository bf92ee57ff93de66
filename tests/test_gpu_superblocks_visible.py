"""Visible-tile lists by way of superblocks, bit for bit against the oracle where their steps change:
candidate rectangles at both sides of the 64 that a mask holds, large ones whose masks are listed, ones
so thin that the list has no room for their superblocks, conics that are not definite or far out of
range (the FP32 tests don't apply), tiles that touch {Q = theta}, few and many ranks, and the largest
superblock grid beside the first that is binned by a sort of the pairs."""
import numpy as np
import pytest
import torch

import oracle
from gpu_util import say, upload
from paper_2604_02120_amd import _lib, api

pytestmark = pytest.mark.gpu


def scene(W, H, n, s_lo, s_hi, seed, aspect=4.0, odd=False, on_grid=False):
    """Ellipses with standard deviations between s_lo and s_hi, the shorter axis up to `aspect` less."""
    rng = np.random.default_rng(seed)
    s1 = np.exp(rng.uniform(np.log(s_lo), np.log(s_hi), n))
    s2 = s1 / rng.uniform(1.0, aspect, n)
    phi = rng.uniform(0.0, np.pi, n)
    c, s = np.cos(phi), np.sin(phi)
    conics = np.stack([c * c / s1**2 + s * s / s2**2, c * s * (1 / s1**2 - 1 / s2**2),
                       s * s / s1**2 + c * c / s2**2], 1).astype(np.float32)
    means = (rng.uniform(-0.1, 1.1, (n, 2)) * [W, H]).astype(np.float32)
    opacity = rng.uniform(0.0, 1.0, n).astype(np.float32) ** 2
    if on_grid:                     # distances and conics whose products are exact
        means = np.floor(means / 8).astype(np.float32) * 8
        conics = np.tile(np.float32([2.0**-6, 0.0, 2.0**-6]), (n, 1))
        opacity[:] = rng.choice(np.float32([1 / 255, 0.5, 1.0]), n)
    if odd:
        k = rng.integers(0, 8, n)
        conics[k == 1] = 0.0
        conics[k == 2, 1] = 1.0
        conics[k == 3, 0] *= -1.0
        conics[k == 4] *= np.float32(1e25)
        conics[k == 5] *= np.float32(1e-25)
        conics[k == 6, 1] = np.sqrt(conics[k == 6, 0] * conics[k == 6, 2])
    return dict(width=W, height=H, means2d=means, conics=conics, opacity=opacity,
                colors=np.zeros((n, 3), np.float32),
                depths=rng.integers(1, 50, n).astype(np.float32),
                radii=np.minimum(np.ceil(3 * s1), 60000).astype(np.int32))


SCENES = {
    "one": lambda: scene(16, 16, 1, 4, 4, 1),
    "masks of 64": lambda: scene(700, 500, 3000, 18, 32, 2),
    "large": lambda: scene(1030, 1000, 1300, 60, 600, 3),
    "thin": lambda: scene(4096, 4096, 200, 1000, 3000, 4, aspect=3000.0),
    "odd conics": lambda: scene(333, 217, 6000, 1, 40, 5, odd=True),
    "on the grid": lambda: scene(640, 480, 5000, 8, 8, 6, on_grid=True),
    "4096 ranks": lambda: scene(300, 200, 4096, 1, 20, 7),
    "131073 ranks": lambda: scene(701, 501, 131073, 1, 6, 8),
    "windows": lambda: scene(2000, 1100, 9000, 1, 300, 9),
    "1024 superblocks": lambda: scene(4096, 4096, 6000, 1, 40, 10),
    "past 1024 superblocks": lambda: scene(4097, 4096, 6000, 1, 40, 11, odd=True),
}


def lists(s, gpu):
    W, H = s["width"], s["height"]
    ref = oracle.bin_tiles(s["means2d"], s["radii"], s["depths"], W, H, s["conics"], s["opacity"],
                                oracle.BIN_VISIBLE)
    return ref, upload(s, gpu)


@pytest.mark.parametrize("name", list(SCENES))
def test_lists_bitexact(gpu, name):
    s = SCENES[name]()
    W, H = s["width"], s["height"]
    say(f"[visible superblocks] {name} {W}x{H} n={len(s['radii'])}")
    (pl_ref, rg_ref), sd = lists(s, gpu)
    pl, rg = api.bin_tiles(sd["means2d"], sd["radii"], sd["depths"], W, H, conics=sd["conics"],
                           opacity=sd["opacity"], mode="visible")
    np.testing.assert_array_equal(rg.cpu().numpy().astype(np.uint32), rg_ref)
    np.testing.assert_array_equal(pl.cpu().numpy().astype(np.uint32), pl_ref)


@pytest.mark.parametrize("name", ["large", "thin"])
def test_fill_repeats_and_overflow_stays_inside(gpu, name):
    """One count serves several fills, with and without room for the list; a capacity below the pair
    count gives the status word and nothing past it."""
    s = SCENES[name]()
    W, H, n = s["width"], s["height"], len(s["radii"])
    (pl_ref, rg_ref), sd = lists(s, gpu)
    pairs = len(pl_ref)
    gx, gy = api.grid(W, H)
    kw = dict(conics=sd["conics"], opacity=sd["opacity"], mode="visible")
    room = 4 * pairs + 400000
    big = api.BinWorkspace(n, room, W, H, device=gpu)
    api.bin_count(sd["means2d"], sd["radii"], W, H, big, **kw)
    for cap, want in ((pairs, _lib.GSB_OK), (room, _lib.GSB_OK), (pairs - 1, _lib.GSB_ERR_CAPACITY),
                      (pairs, _lib.GSB_OK), (1, _lib.GSB_ERR_CAPACITY)):
        pl = torch.full((room + 64,), -7, dtype=torch.int32, device=gpu)
        rg = torch.full((gx * gy, 2), -1, dtype=torch.int32, device=gpu)
        st = api.bin_fill(sd["means2d"], sd["radii"], sd["depths"], W, H, big, pl[:cap], rg, **kw)
        assert int(st.item()) == want
        assert bool((pl[cap:] == -7).all())
        assert 0 <= int(rg.min()) and int(rg.max()) <= cap
        if want == _lib.GSB_OK:
            np.testing.assert_array_equal(pl[:pairs].cpu().numpy().astype(np.uint32), pl_ref)
            np.testing.assert_array_equal(rg.cpu().numpy().astype(np.uint32), rg_ref)
