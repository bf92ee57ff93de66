"""Tile lists of few Gaussians, bit for bit against the oracle, at the edges of what is written in one
launch: one chunk of 64 ranks, ragged chunks, the most Gaussians and the first past them, the widest
grid of 128 tile columns beside the first past it, and the most cells; and of the most that are
ranked by counting (16384) beside the first past them."""
import numpy as np
import pytest
import torch

import oracle
from gpu_util import say, upload
from paper_2604_02120_amd import _lib, api
from test_gpu_superblocks import scene

pytestmark = pytest.mark.gpu

SCENES = {
    "one chunk": (64, 64, 64, 0, 40),
    "65 ranks": (64, 64, 65, 0, 40),
    "1087 ranks, ragged grid": (333, 217, 1087, 0, 300),
    "4096 ranks on every tile": (200, 136, 4096, 300, 400),
    "4097 ranks": (200, 136, 4097, 0, 90),
    "128 columns": (2048, 1120, 3000, 0, 500),
    "129 columns": (2049, 1120, 3000, 0, 500),
    "129 columns, 1000 ranks": (2049, 200, 1000, 0, 500),
    "129 columns, 2000 ranks": (2049, 200, 2000, 0, 500),
    "128 rows": (1120, 2048, 3000, 0, 500),
    "more cells": (1150, 2048, 3000, 0, 500),
    "one column": (10, 2048, 900, 1, 200),
    "63 ranks": (100, 90, 63, 0, 40),
    "8191 ranks": (400, 300, 8191, 0, 30),
    "16384 ranks": (400, 300, 16384, 0, 30),
    "16385 ranks": (400, 300, 16385, 0, 30),
}


@pytest.mark.parametrize("name", list(SCENES))
def test_lists_bitexact(gpu, name):
    W, H, n, lo, hi = SCENES[name]
    s = scene(W, H, n, lo, hi, 31, levels=9)
    say(f"[few lists] {name} {W}x{H} n={n}")
    pl_ref, rg_ref = oracle.bin_tiles(s["means2d"], s["radii"], s["depths"], W, H)
    sd = upload(s, gpu)
    pl, rg = api.bin_tiles(sd["means2d"], sd["radii"], sd["depths"], W, H)
    np.testing.assert_array_equal(rg.cpu().numpy().astype(np.uint32), rg_ref)
    np.testing.assert_array_equal(pl.cpu().numpy().astype(np.uint32), pl_ref)


def test_overflow_stays_inside(gpu):
    s = scene(333, 217, 1087, 0, 300, 31, levels=9)
    W, H, n = 333, 217, 1087
    pl_ref, rg_ref = oracle.bin_tiles(s["means2d"], s["radii"], s["depths"], W, H)
    pairs = len(pl_ref)
    sd = upload(s, gpu)
    gx, gy = api.grid(W, H)
    ws = api.BinWorkspace(n, pairs, W, H, device=gpu)
    api.bin_count(sd["means2d"], sd["radii"], W, H, ws)
    for cap, want in ((pairs - 1, _lib.GSB_ERR_CAPACITY), (pairs, _lib.GSB_OK)):
        pl = torch.full((pairs + 64,), -7, dtype=torch.int32, device=gpu)
        rg = torch.full((gx * gy, 2), -1, dtype=torch.int32, device=gpu)
        st = api.bin_fill(sd["means2d"], sd["radii"], sd["depths"], W, H, ws, pl[:cap], rg)
        assert int(st.item()) == want
        assert bool((pl[cap:] == -7).all())
        assert 0 <= int(rg.min()) and int(rg.max()) <= cap
    np.testing.assert_array_equal(pl[:pairs].cpu().numpy().astype(np.uint32), pl_ref)
    np.testing.assert_array_equal(rg.cpu().numpy().astype(np.uint32), rg_ref)
