"""bin_tiles on a stream that is not the current one: its scratch and its results come from that stream's
memory (the current stream's is left as it was), so that work enqueued on the current stream meanwhile
cannot be given what the binning's kernels still use. For frames with fewer pairs than the first
workspace holds, and with more, in both modes; against the oracle bit for bit."""
import numpy as np
import pytest
import torch

import oracle
from gpu_util import say, upload
from paper_2604_02120_amd import api

pytestmark = pytest.mark.gpu


def segments(stream) -> list:
    """(address, size) of the memory held for a stream."""
    return sorted((s["address"], s["total_size"]) for s in torch.cuda.memory_snapshot()
                  if s["stream"] == stream.cuda_stream)


def holds(stream, t) -> bool:
    return any(a <= t.data_ptr() < a + size for a, size in segments(stream))


@pytest.mark.parametrize("external", [False, True])
@pytest.mark.parametrize("mode", ["rect", "visible"])
@pytest.mark.parametrize("name,n,radius", [("within the guess", 30000, 9), ("past it", 20000, 70)])
def test_other_stream(gpu, name, n, radius, mode, external):
    say(f"[bin stream] {name} {mode} external={external}")
    W, H = 640, 480
    rng = np.random.default_rng(n)
    s = dict(width=W, height=H, means2d=(rng.uniform(0, 1, (n, 2)) * [W, H]).astype(np.float32),
             opacity=rng.uniform(0.01, 1.0, n).astype(np.float32),
             colors=rng.uniform(0, 1, (n, 3)).astype(np.float32),
             depths=rng.uniform(1, 9, n).astype(np.float32), radii=np.full(n, radius, np.int32))
    i2 = np.full(n, (radius / 3.0) ** -2, np.float32)
    s["conics"] = np.stack([i2, np.float32(0.3) * i2, i2], 1)
    vis = dict(conics=s["conics"], opacity=s["opacity"], mode=oracle.BIN_VISIBLE) if mode == "visible" else {}
    pl_ref, rg_ref = oracle.bin_tiles(s["means2d"], s["radii"], s["depths"], W, H, **vis)
    assert mode == "visible" or (len(pl_ref) > api._GUESS * n) == (name == "past it")
    sd = upload(s, gpu)
    side = torch.cuda.Stream()
    given = torch.cuda.ExternalStream(side.cuda_stream) if external else side
    cur = torch.cuda.current_stream()
    vis = dict(conics=sd["conics"], opacity=sd["opacity"], mode="visible") if mode == "visible" else {}
    api.bin_tiles(sd["means2d"], sd["radii"], sd["depths"], W, H, **vis)      # (code is loaded)
    torch.cuda.synchronize()
    torch.cuda.empty_cache()
    before = segments(cur)
    outs = []
    for _ in range(3):
        pl, rg = api.bin_tiles(sd["means2d"], sd["radii"], sd["depths"], W, H, stream=given, **vis)
        assert segments(cur) == before
        assert holds(side, rg) and (not len(pl_ref) or holds(side, pl))
        outs.append((pl, rg))
    # what the current stream is given now is written while the binning may still run
    junk = [torch.full((1 << 20,), -1, dtype=torch.int32, device=gpu) for _ in range(8)]
    cur.wait_stream(side)
    for pl, rg in outs:
        np.testing.assert_array_equal(rg.cpu().numpy().astype(np.uint32), rg_ref)
        np.testing.assert_array_equal(pl.cpu().numpy().astype(np.uint32), pl_ref)
    assert all(bool((j == -1).all()) for j in junk)
