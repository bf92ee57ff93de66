"""A binning workspace serves every list up to its capacity: its size never falls as the capacity
grows, also where the chunks of the superblock entries change their length."""
import pytest

from paper_2604_02120_amd import _lib


@pytest.mark.parametrize("n", [1, 2000, 32768, 40000, 49152, 300000])
def test_size_grows_with_capacity(n):
    caps = [0, 1, 255, 256, 1024] + [(1 << 19) + d for d in (-1, 0, 1, 1000, 11000, 1 << 19)] + [1 << 21]
    sizes = [_lib.gsb_bin_workspace_bytes(n, c, 640, 480) for c in caps]
    assert sizes == sorted(sizes), list(zip(caps, sizes))
