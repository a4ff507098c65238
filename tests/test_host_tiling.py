"""The tiling of a small call, as the host-only plan describes it: the whole
LDS and 1024 threads, asked for with the largest tile_px."""

import pytest

from paper_2209_13168_amd import ecmd
from tests.test_host_plan import SENSORS


@pytest.mark.parametrize("W,H,foe", SENSORS[:4])
@pytest.mark.parametrize("pol", [False, True])
def test_whole_lds_tiles(W, H, foe, pol):
    p = ecmd.plan(ecmd.sensor(W, H, foe), 0.0, 1.5, 1e-5, polarity=pol, tile_px=2**31 - 1)
    tiles = {128: 4, 346: 4, 640: 8, 1280: 24}[W]
    assert (p["segments"], p["eval_threads"]) == (tiles * (2 if pol else 1), 1024)
    # the counters and the kernel's 420 bytes beside them, in whole 16 bytes
    assert p["tile_budget_px"] == (160 * 1024 - 420) // 16 * 4
