"""Event binning at the edges of its chunks and of the counter scan: window
sizes around a chunk, totals on both sides of the line between the two
workgroup sizes, and enough windows for several rounds of the scan."""

import numpy as np
import pytest

from synth import pack_batch
from synth.ventral import WindowSpec, make_window

pytestmark = pytest.mark.gpu

FEW = 1 << 22  # events from which the large workgroups take over


@pytest.fixture(scope="module")
def ctx():
    from paper_2209_13168_amd import ecmd

    with ecmd.Context(0) as c:
        yield c


@pytest.mark.parametrize("n", [1, 1023, 1024, 1025, FEW - 1, FEW, FEW + 4097])
def test_probe_at_the_chunk_edges(ctx, n):
    """Sums of squares and counts are whole numbers: equal to the oracle's."""
    from oracle import oracle as O
    from paper_2209_13168_amd import ecmd

    rng = np.random.default_rng(n)
    W, H, tau, foe = 346, 260, 0.25, (170.25, 131.5)
    x = rng.uniform(-3, W + 3, n).astype(np.float32)
    y = rng.uniform(-3, H + 3, n).astype(np.float32)
    t = np.sort(rng.uniform(0, tau, n)).astype(np.float32)
    ev = O.Events(x, y, t, tau, W, H, foe)
    sen = ecmd.sensor(W, H, foe)
    ds = np.array([0.0, 0.31, 1.9], np.float32)
    S, N = ctx.probe_point(sen, x, y, t, tau, ds)[:2]
    for k, d in enumerate(ds):
        assert (int(S[k]), int(N[k])) == O.point(ev, float(d))[:2]
    S, N = ctx.probe_bound(sen, x, y, t, tau, 0.0, 2.0, ds[:-1], ds[1:])[:2]
    for k in range(2):
        assert (int(S[k]), int(N[k])) == O.bound(ev, float(ds[k]), float(ds[k + 1]))[:2]


def test_many_windows_scan_in_several_rounds(ctx):
    """400 windows: more counters than one round of the scan takes."""
    from oracle import oracle as O
    from paper_2209_13168_amd import ecmd

    spec = WindowSpec(width=128, height=128, foe=(63.3, 61.8), tau=0.2, n_events=60, d_true=0.7, n_points=20,
                      noise_frac=0.2, d_lo=0.0, d_hi=2.0,
                      eps=1e-2)
    wins = [make_window(spec, 0, k) for k in range(400)]
    res = ctx.estimate_batched(ecmd.sensor(128, 128, spec.foe), *pack_batch(wins), spec.d_lo, spec.d_hi, spec.eps)
    for k in [0, 1, 170, 171, 341, 342, 398, 399]:
        o = O.bnb(O.Events.of_window(wins[k]), spec.d_lo, spec.d_hi, spec.eps)
        assert (res[k].status, res[k].j_star, res[k].K) == (0, o.j_star, o.K), k
