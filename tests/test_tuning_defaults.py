"""A tuning dict that names some fields leaves the others as they are without a tuning: the launch too,
which is 0 (persistent) in a zeroed struct but the library's choice (a block per item) without one."""
import pytest

from paper_2604_02120_amd import _lib, api, autotune


@pytest.mark.parametrize("given,launch", [
    (None, None), ({}, None), ({"batch_bwd": 128}, _lib.GSB_LAUNCH_GRID),
    ({"batch_fwd": 64, "launch": 0}, _lib.GSB_LAUNCH_PERSISTENT), ({"launch": 1}, _lib.GSB_LAUNCH_GRID),
    ({"blocks_per_cu": 2}, _lib.GSB_LAUNCH_PERSISTENT)])
def test_launch(monkeypatch, given, launch):
    seen = []
    monkeypatch.setattr(_lib, "gsb_plan_create", lambda views, prec, t: seen.append(t))
    bv = api.BatchedViews.__new__(api.BatchedViews)
    bv.plan, bv.views, bv.prec = None, [], 0
    bv._make_plan(given)
    assert (seen[0] is None) == (launch is None)
    if launch is not None:
        assert seen[0].launch == launch
        assert seen[0].batch_fwd == given.get("batch_fwd", 0) and seen[0].batch_bwd == given.get("batch_bwd", 0)


def test_saved_tunings_name_the_launch():
    assert all(set(c) == set(autotune.KEYS) for c in autotune.CANDIDATES)
