"""Calls of few events whose items leave most of the chip empty take the
tiles of larger calls: single large windows of a sensor cut three times as
fine, probes of few intervals.  On both sides of each line the results are
those of forced tiles and workgroups, field by field, and the oracle's."""

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

SENSORS = {(640, 480): (320.0, 240.0), (346, 260): (173.0, 130.0)}
TAU = 0.25


def _window(W, H, foe, n, seed):
    rng = np.random.default_rng(seed)
    # points that move away from the FOE at divergence 0.7, and noise
    x0, y0 = rng.uniform(0, W, 5000), rng.uniform(0, H, 5000)
    k = rng.integers(0, 5000, n)
    t = np.sort(rng.uniform(0, TAU, n)).astype(np.float32)
    r = 0.7 / (1.0 - 0.7 * TAU)
    s = 1.0 / (1.0 + r * (TAU - t))
    x = (foe[0] + (x0[k] - foe[0]) * s).astype(np.float32)
    y = (foe[1] + (y0[k] - foe[1]) * s).astype(np.float32)
    noise = rng.random(n) < 0.1
    x[noise] = rng.uniform(0, W, noise.sum()).astype(np.float32)
    return x, y, t


@pytest.fixture(scope="module")
def ctx():
    from paper_2209_13168_amd import ecmd

    c = ecmd.Context(0)
    yield c
    c.close()


def _forced(ctx, run):
    got = run()
    saved = ctx.tuning()
    try:
        for tile_px, nt in ((13000, 512), (40000, 1024)):
            ctx.set_tuning(tile_px=tile_px, eval_threads=nt)
            other = run()
            for g, o in zip(got, other):
                assert np.array_equal(g, o) if isinstance(g, np.ndarray) else g == o, (tile_px, nt)
    finally:
        ctx.set_tuning(**saved)
    return got


@pytest.mark.parametrize("sizes", [[599_999], [600_000], [900_000, 299_999], [900_000, 300_000]],
                         ids=lambda s: "-".join(map(str, s)))
@pytest.mark.parametrize("W,H", SENSORS)
def test_windows(ctx, orc, W, H, sizes):
    from paper_2209_13168_amd import ecmd

    foe = SENSORS[W, H]
    wins = [_window(W, H, foe, n, 3 + k) for k, n in enumerate(sizes)]
    x, y, t = (np.concatenate(a) for a in zip(*wins))
    off = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int64)
    tau = np.full(len(sizes), TAU, np.float32)
    got = _forced(ctx, lambda: ctx.estimate_batched(ecmd.sensor(W, H, foe), x, y, t, off, tau, 0.0, 1.5, 1e-4))
    for (wx, wy, wt), r in zip(wins, got):
        S, N = orc.point(orc.Events(wx, wy, wt, TAU, W, H, foe), float(r.d_hat))[:2]
        assert r.status == 0 and r.K == W * H * S - N * N


@pytest.mark.parametrize("n,m", [(299_999, 4), (300_000, 1), (300_000, 16), (300_000, 17)])
@pytest.mark.parametrize("W,H", SENSORS)
def test_probes(ctx, orc, W, H, n, m):
    from paper_2209_13168_amd import ecmd

    foe = SENSORS[W, H]
    x, y, t = _window(W, H, foe, n, 11)
    e = np.linspace(0.1, 1.2, m + 1).astype(np.float32)
    sen = ecmd.sensor(W, H, foe)
    S, N = _forced(ctx, lambda: ctx.probe_bound(sen, x, y, t, TAU, 0.0, 1.5, e[:-1].copy(), e[1:].copy())[:2])
    ev = orc.Events(x, y, t, TAU, W, H, foe)
    for k in {0, m - 1}:
        assert (int(S[k]), int(N[k])) == tuple(orc.bound(ev, float(e[k]), float(e[k + 1]))[:2])
