"""A plan whose caller limits the event records accepts what it accepted on
the tiles of a large call, whatever the tiles of a small one: events that
cross a cut of the whole-LDS tiles but none of the finer ones, with room for
one record each."""

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("room", [0, 4000, 7999, 8000])  # records; 0: the default
def test_own_record_limit(room):
    import torch

    from paper_2209_13168_amd import ecmd

    W, H, foe, tau, n = 640, 480, (320.0, 240.0), 0.25, 4000
    sen = ecmd.sensor(W, H, foe)
    fine, whole = ecmd.plan(sen, 0.0, 1.5, 1e-4), ecmd.plan(sen, 0.0, 1.5, 1e-4, tile_px=1 << 30)
    assert 160 in whole["colcut"] and 160 not in fine["colcut"]
    r = np.random.default_rng(1)
    # up to 20 ms before the window's end: they move less than 10 pixels
    x = r.uniform(155, 170, n).astype(np.float32)
    y = r.uniform(50, 80, n).astype(np.float32)
    t = np.sort(r.uniform(tau - 0.02, tau, n)).astype(np.float32)
    a = (x - 320) * (tau - t)
    over = (x >= 160) & (x + a * 2.4 < 160)
    assert over.sum() > 100 and (x - 8 > max(c for c in fine["colcut"] if c < 160)).all()
    off, ta = np.array([0, n], np.int64), np.array([tau], np.float32)
    with ecmd.Context(0) as ctx:
        want = ctx.estimate_batched(sen, x, y, t, off, ta, 0.0, 1.5, 1e-4)
        plan = ctx.batch_plan(sen, 0.0, 1.5, 1e-4, 1, n, max_records=room)
        out = plan.result_buffer(1)
        plan.launch(*(torch.from_numpy(v).cuda() for v in (x, y, t, off, ta)), out)
        torch.cuda.synchronize()
        assert plan.results(out, 1) == want and want[0].status == 0
