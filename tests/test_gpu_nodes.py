"""Node groups (k_nodes): neighbouring nodes evaluated from one image.

Groups form only when a launch holds many (window, tile) segments, so a batch
of small-sensor windows uses them where the same windows one per call are
evaluated hypothesis by hypothesis; every field of the results (counters
included) must agree, and the optimum must be the oracle's.  The cases put
segments at the edges of waves and chunks, fill one strip of a tile, outgrow
the lists, use a sensor without integer FOE (guest copies) and both images of
the polarity-aware contrast."""

import dataclasses

import numpy as np
import pytest

from synth import config_windows, pack_batch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    from paper_2209_13168_amd import ecmd

    c = ecmd.Context(0)
    yield c
    c.close()


def _run(ctx, wins, foe=None, pol=False, **kw):
    from paper_2209_13168_amd import ecmd

    s = wins[0].spec
    x, y, t, off, tau = pack_batch(wins)
    p = np.concatenate([w.p for w in wins]) if pol else None
    return ctx.estimate_batched(ecmd.sensor(s.width, s.height, foe or s.foe), x, y, t, off, tau, s.d_lo, s.d_hi, s.eps,
                                polarity=p, **kw)


def _same(ctx, orc, wins, foe=None, pol=False, check=2, **kw):
    assert len(wins) >= 8
    got = _run(ctx, wins, foe, pol, **kw)
    alone = [_run(ctx, [w], foe, pol, **kw)[0] for w in wins]
    assert got == alone
    for w, r in list(zip(wins, got))[:check]:
        s = w.spec
        if pol:
            continue
        o = orc.bnb(orc.Events(w.x, w.y, w.t_rel, np.float32(s.tau), s.width, s.height, foe or s.foe), s.d_lo, s.d_hi,
                    s.eps)
        assert (r.j_star, r.K) == (o.j_star, o.K)
    return got


@pytest.mark.parametrize("n", [1, 63, 64, 65, 511, 513, 2049, 9000])
def test_segment_sizes(ctx, orc, n):
    _same(ctx, orc, config_windows("c1", range(8), n_events=n, n_points=max(1, n // 30)))


@pytest.mark.parametrize("foe", [(173.0, 130.0), (101.3, 57.85)])
def test_tiles_and_guests(ctx, orc, foe):
    wins = config_windows("c2", range(8), n_events=9000)
    _same(ctx, orc, [dataclasses.replace(w, spec=dataclasses.replace(w.spec, eps=1e-4)) for w in wins], foe=foe, check=1)


def test_polarity(ctx, orc):
    _same(ctx, orc, config_windows("c1", range(8), n_events=6000), pol=True)


def _placed(n, seed, xs, ys, ts):
    """Windows of the 128x128 sensor with events drawn from the given ranges."""
    out = []
    for k, w in enumerate(config_windows("c1", range(8), n_events=8)):
        r = np.random.default_rng(seed + k)
        u = [r.uniform(*lim, n).astype(np.float32) for lim in (xs, ys, ts)]
        out.append(dataclasses.replace(w, x=u[0], y=u[1], t_rel=np.sort(u[2]), p=np.ones(n, np.int8),
                                       owner=np.full(n, -1, np.int32)))
    return out


@pytest.mark.parametrize("name,n,xs,ys,ts", [
    ("corner", 60_000, (118, 120), (118, 120), (0.0, 0.001)),  # four times the mean motion: the lists are outgrown
    ("row", 20_000, (64, 127), (70, 71), (0.0, 0.4)),          # one strip of a tile
    ("still", 5_000, (63.9, 64.1), (63.9, 64.1), (0.0, 0.4)),  # nothing moves
    ("last", 5_000, (0, 127), (0, 127), (0.499, 0.4999)),      # at the window's end
])
def test_placed_events(ctx, orc, name, n, xs, ys, ts):
    _same(ctx, orc, _placed(n, 5, xs, ys, ts), check=1)


def test_budgets_and_policies(ctx, orc):
    wins = config_windows("c1", range(8), n_events=4000)
    _same(ctx, orc, wins, check=0, max_nodes=37)
    _same(ctx, orc, wins, frontier_batch=7)
    _same(ctx, orc, wins, frontier_batch=1024)
    _same(ctx, orc, wins, exact_bounds=True)
    _same(ctx, orc, wins, check=0, gamma=0.01)


def test_lists_of_the_allocation_free_call(ctx):
    """The static scratch leaves the lists what the other buffers do not
    need: ample, short, or none; the results do not change."""
    import torch

    from paper_2209_13168_amd import ecmd

    wins = config_windows("c1", range(8), n_events=4000)
    s = wins[0].spec
    want = _run(ctx, wins)
    args = [torch.from_numpy(a).cuda() for a in pack_batch(wins)]
    out = ecmd.BatchPlan.result_buffer(8)
    for cap, most in ((2048, 40_000), (16384, 1_000_000), (16384, 3_500_000)):
        out.zero_()
        ctx.estimate_batched_noalloc(ecmd.sensor(s.width, s.height, s.foe), *args, s.d_lo, s.d_hi, s.eps, most, out,
                                     frontier_capacity=cap)
        torch.cuda.synchronize()
        assert ecmd.BatchPlan.results(out, 8) == want


@pytest.mark.parametrize("n", [24 * 128 * 128, 24 * 128 * 128 + 1])
def test_dense_small_windows(ctx, orc, n):
    """Both sides of the line above which a small image's windows form no groups."""
    from paper_2209_13168_amd import ecmd

    wins = _placed(n, 9, (40, 90), (40, 90), (0.0, 0.4))[:2]
    s = wins[0].spec
    got = _run(ctx, wins)
    saved = ctx.tuning()
    try:
        ctx.set_tuning(tile_px=6000, eval_threads=256)
        assert _run(ctx, wins) == got
    finally:
        ctx.set_tuning(**saved)
    S, N = ctx.probe_point(ecmd.sensor(s.width, s.height, s.foe), wins[0].x, wins[0].y, wins[0].t_rel, s.tau,
                           np.array([got[0].d_hat], np.float32))[:2]
    ev = orc.Events(wins[0].x, wins[0].y, wins[0].t_rel, np.float32(s.tau), s.width, s.height, s.foe)
    So, No = orc.point(ev, float(got[0].d_hat))[:2]
    assert (int(S[0]), int(N[0])) == (So, No) and got[0].K == s.width * s.height * So - No * No
