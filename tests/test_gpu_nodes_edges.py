"""Node groups against searches that form none: the allocation-free call forms
groups with the lists that its scratch leaves room for, and none where that is
less than 64 events a wave, so one batch is searched with lists of every
length and without."""

import numpy as np
import pytest

from synth import config_windows, pack_batch
from tests.test_gpu_nodes import _placed, _run

pytestmark = pytest.mark.gpu

MIB = 1 << 20
LISTS = 32 * 16 * 256  # bytes of all lists per event of a wave's (16 waves on 256 CUs)


@pytest.fixture(scope="module")
def ctx():
    from paper_2209_13168_amd import ecmd

    c = ecmd.Context(0)
    yield c
    c.close()


def _noalloc(ctx, wins, cap):
    """The batch with lists of `cap` events a wave (0: no groups): what is left
    of the scratch after the frontier, which takes the rest."""
    import torch

    from paper_2209_13168_amd import ecmd

    s, B = wins[0].spec, len(wins)
    arrs = pack_batch(wins)
    n = int(arrs[3][-1])
    # room for lists of `cap` events and half as many again: not for twice
    room = LISTS * (cap + cap // 2 if cap else 32)
    fixed = 16 * (n + 2048) + 3 * MIB  # the event store and the small buffers
    capacity = (64 * MIB - room - fixed) // (32 * B)
    out = ecmd.BatchPlan.result_buffer(B)
    args = [torch.from_numpy(a).cuda() for a in arrs]
    ctx.estimate_batched_noalloc(ecmd.sensor(s.width, s.height, s.foe), *args, s.d_lo, s.d_hi, s.eps, n, out,
                                 frontier_capacity=capacity)
    torch.cuda.synchronize()
    return ecmd.BatchPlan.results(out, B)


# "corner": whole points of events at four times the mean motion cross pixel
# edges together and outgrow the lists (counted in an instrumented kernel: 21 of
# 41 groups and tiles with lists of 64, 61 of 81 with 128, 113 of 154 with 256,
# 346 of 484 with 1024; none in the others)
CASES = {
    "descent": lambda: config_windows("c1", range(8), n_events=20_000),
    "corner": lambda: _placed(60_000, 5, (118, 120), (118, 120), (0.0, 0.001)),
    "corners": lambda: _placed(60_000, 5, (100, 127), (100, 127), (0.0, 0.4)),
    "dense": lambda: _placed(24 * 128 * 128, 9, (40, 90), (40, 90), (0.0, 0.4))[:2],
}


@pytest.mark.parametrize("case", CASES)
def test_lists_of_every_length(ctx, case):
    wins = CASES[case]()
    want = _noalloc(ctx, wins, 0)
    assert all(r.status == 0 for r in want)
    for cap in (64, 128, 256):
        assert _noalloc(ctx, wins, cap) == want, cap
    assert _run(ctx, wins) == want  # 1024
