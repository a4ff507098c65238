"""Calls of few events take whole-LDS tiles and the largest workgroups, and
one window of many events is evaluated in node groups; at both sides of both
lines every field of the result is what forced tiles and workgroups give, and
the optimum's key is the oracle's at that divergence."""

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [299_999, 300_000, 3_499_999, 3_500_000])
@pytest.mark.parametrize("pol", [False, True])
def test_lines_between_the_rules(n, pol):
    from oracle import oracle as O
    from paper_2209_13168_amd import ecmd

    W, H, tau, foe = 346, 260, 0.25, (173.0, 130.0)
    rng = np.random.default_rng(n)
    # points that move away from the FOE at divergence 0.8, and noise
    x0, y0 = rng.uniform(0, W, 4000), rng.uniform(0, H, 4000)
    k = rng.integers(0, 4000, n)
    t = np.sort(rng.uniform(0, tau, n)).astype(np.float32)
    r = 0.8 / (1.0 - 0.8 * tau)
    s = 1.0 / (1.0 + r * (tau - t))
    x = (foe[0] + (x0[k] - foe[0]) * s).astype(np.float32)
    y = (foe[1] + (y0[k] - foe[1]) * s).astype(np.float32)
    noise = rng.random(n) < 0.1
    x[noise] = rng.uniform(0, W, noise.sum()).astype(np.float32)
    p = rng.choice(np.array([-1, 1], np.int8), n) if pol else None
    off, ta = np.array([0, n], np.int64), np.array([tau], np.float32)
    with ecmd.Context(0) as ctx:
        run = lambda: ctx.estimate_batched(ecmd.sensor(W, H, foe), x, y, t, off, ta, 0.0, 2.0, 1e-4, polarity=p)[0]
        got = run()
        ctx.set_tuning(tile_px=13000, eval_threads=512)
        assert run() == got
    assert got.status == 0
    ev = O.Events(x, y, t, tau, W, H, foe, p) if pol else O.Events(x, y, t, tau, W, H, foe)
    S, N = (O.point_pol if pol else O.point)(ev, float(got.d_hat))[:2]
    M = W * H * (2 if pol else 1)
    assert got.K == M * S - N * N
