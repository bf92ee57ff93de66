"""Tile lists by way of superblocks of 8 x 8 tiles, bit for bit against the oracle at the sizes where
their steps change: one Gaussian, partial superblocks, several chunks of 1024 entries in one
superblock, lists that go through LDS in parts, more entries per block than are ranked at a time,
and the largest grids (1024 superblocks) beside the first that is binned by a sort of the pairs."""
import numpy as np
import pytest
import torch

import oracle
from gpu_util import say, upload
from paper_2604_02120_amd import _lib, api

pytestmark = pytest.mark.gpu


def scene(W, H, n, r_lo, r_hi, seed, levels=None):
    rng = np.random.default_rng(seed)
    depths = rng.uniform(1.0, 100.0, n).astype(np.float32)
    if levels:
        depths = np.floor(depths / 100.0 * levels).astype(np.float32) + 1.0
    return dict(width=W, height=H,
                means2d=(rng.uniform(-0.1, 1.1, (n, 2)) * [W, H]).astype(np.float32),
                conics=np.tile(np.float32([1.0, 0.0, 1.0]), (n, 1)),
                opacity=np.full(n, 0.5, np.float32), colors=np.zeros((n, 3), np.float32),
                depths=depths, radii=rng.integers(r_lo, r_hi + 1, n).astype(np.int32))


SCENES = {
    "one": lambda: scene(16, 16, 1, 8, 8, 1),
    "none visible": lambda: scene(40, 24, 300, 0, 0, 2),
    "one superblock, every tile": lambda: scene(128, 128, 3000, 400, 500, 3, levels=5),
    "partial superblocks": lambda: scene(131, 1035, 4097, 0, 90, 4),
    "quarters of a chunk": lambda: scene(128, 128, 2500, 40, 70, 5),
    "one column": lambda: scene(7, 3000, 5000, 1, 300, 6),
    "windows": lambda: scene(1030, 1000, 1300, 1500, 2000, 7, levels=3),
    "1025 ranks": lambda: scene(300, 200, 1025, 0, 60, 12),
    "2049 ranks": lambda: scene(300, 200, 2049, 0, 60, 13),
    "4096 ranks": lambda: scene(300, 200, 4096, 0, 60, 14, levels=7),
    "131073 ranks": lambda: scene(700, 500, 131073, 0, 12, 15, levels=100),
    "many ranks": lambda: scene(4200, 2100, 30000, 0, 20, 8),        # 561 superblocks
    "wide": lambda: scene(65536, 16, 9000, 0, 700, 9),               # 512 x 1
    "1024 superblocks": lambda: scene(4096, 4096, 6000, 0, 120, 10),
    "past 1024 superblocks": lambda: scene(4097, 4096, 6000, 0, 120, 11),
}


@pytest.mark.parametrize("name", list(SCENES))
def test_lists_bitexact(gpu, name):
    s = SCENES[name]()
    W, H = s["width"], s["height"]
    say(f"[superblocks] {name} {W}x{H} n={len(s['radii'])}")
    pl_ref, rg_ref = oracle.bin_tiles(s["means2d"], s["radii"], s["depths"], W, H)
    sd = upload(s, gpu)
    pl, rg = api.bin_tiles(sd["means2d"], sd["radii"], sd["depths"], W, H)
    np.testing.assert_array_equal(rg.cpu().numpy().astype(np.uint32), rg_ref)
    np.testing.assert_array_equal(pl.cpu().numpy().astype(np.uint32), pl_ref)


def test_fill_repeats_and_overflow_stays_inside(gpu):
    """One count serves several fills; a capacity below the pair count gives the status word and
    ranges inside the capacity, and nothing is written past it."""
    s = SCENES["partial superblocks"]()
    W, H, n = s["width"], s["height"], len(s["radii"])
    pl_ref, rg_ref = oracle.bin_tiles(s["means2d"], s["radii"], s["depths"], W, H)
    pairs = len(pl_ref)
    sd = upload(s, gpu)
    gx, gy = api.grid(W, H)
    big = api.BinWorkspace(n, pairs, W, H, device=gpu)
    api.bin_count(sd["means2d"], sd["radii"], W, H, big)
    for cap, want in ((pairs, _lib.GSB_OK), (pairs - 1, _lib.GSB_ERR_CAPACITY),
                      (pairs, _lib.GSB_OK), (1, _lib.GSB_ERR_CAPACITY)):
        pl = torch.full((pairs + 64,), -7, dtype=torch.int32, device=gpu)
        rg = torch.full((gx * gy, 2), -1, dtype=torch.int32, device=gpu)
        st = api.bin_fill(sd["means2d"], sd["radii"], sd["depths"], W, H, big, pl[:cap], rg)
        assert int(st.item()) == want
        assert bool((pl[cap:] == -7).all())
        assert 0 <= int(rg.min()) and int(rg.max()) <= cap
        if want == _lib.GSB_OK:
            np.testing.assert_array_equal(pl[:cap].cpu().numpy().astype(np.uint32), pl_ref)
            np.testing.assert_array_equal(rg.cpu().numpy().astype(np.uint32), rg_ref)
