"""Node groups on grids so deep that neighbouring grid points share a rate,
with few nodes a step, so that nodes wait in the queue while their neighbours'
children are queued behind them: the same windows one per call are evaluated
hypothesis by hypothesis, and the optimum is the oracle's."""

import dataclasses

import numpy as np
import pytest

from synth import config_windows
from tests.test_gpu_nodes import _same

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    from paper_2209_13168_amd import ecmd

    c = ecmd.Context(0)
    yield c
    c.close()


def _wins(L, n, d_hi):
    out = []
    for w in config_windows("c1", range(8), n_events=n):
        s = dataclasses.replace(w.spec, eps=d_hi * 2.0 ** -L, d_lo=0.0, d_hi=d_hi)
        out.append(dataclasses.replace(w, spec=s))
    return out


@pytest.mark.parametrize("L", [25, 27, 28, 30])
@pytest.mark.parametrize("F", [2, 3, 16, 0])
def test_deep_grids(ctx, orc, L, F):
    from paper_2209_13168_amd import ecmd

    wins = _wins(L, 1500, 1.5)
    s = wins[0].spec
    assert ecmd.plan(ecmd.sensor(s.width, s.height, s.foe), s.d_lo, s.d_hi, s.eps)["L"] == L
    # neighbouring grid points of one rate, in 32 bits as the search computes it
    tau = np.float32(s.tau)
    rate = [(d := np.float32(ecmd.grid_point(s.d_lo, s.d_hi, L, j))) / (np.float32(1) - d * tau)
            for j in range((1 << L) * 3 // 4, (1 << L) * 3 // 4 + 64)]
    assert L < 27 or len(set(rate)) < len(rate)
    _same(ctx, orc, wins, check=1, frontier_batch=F)


@pytest.mark.parametrize("budget", [60, 90, 200])
def test_deep_grids_cut_short(ctx, orc, budget):
    _same(ctx, orc, _wins(28, 1500, 1.5), check=0, frontier_batch=5, max_nodes=budget)
