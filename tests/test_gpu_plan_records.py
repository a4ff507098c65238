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


def _crossing(n, W=640, H=480):
    """Events that reach four of the finer tiles and one of the whole-LDS ones."""
    r = np.random.default_rng(2)
    x, y = r.uniform(220, 230, n).astype(np.float32), r.uniform(125, 135, n).astype(np.float32)
    return x, y, np.sort(r.uniform(0, 0.01, n)).astype(np.float32)


def test_a_limit_that_holds_every_copy_of_the_coarse_tiles():
    """One window of 700k events, which takes finer tiles by itself."""
    import torch

    from paper_2209_13168_amd import ecmd

    sen, n, tau = ecmd.sensor(640, 480, (320.0, 240.0)), 700_000, 0.25
    arrs = (*_crossing(n), np.array([0, n], np.int64), np.array([tau], np.float32))
    dev = [torch.from_numpy(v).cuda() for v in arrs]
    with ecmd.Context(0) as ctx:
        want = ctx.estimate_batched(sen, *arrs, 0.0, 1.5, 1e-4)
        for room in (0, 2 * n):
            plan = ctx.batch_plan(sen, 0.0, 1.5, 1e-4, 1, n, max_records=room)
            out = plan.result_buffer(1)
            plan.launch(*dev, out)
            torch.cuda.synchronize()
            assert plan.results(out, 1) == want and want[0].status == 0, room


@pytest.mark.parametrize("n", [600_000, 1_000_000])
def test_the_scratch_holds_the_coarse_tiles_records(n):
    """The allocation-free call's event store: 96 bytes an event on the finer
    tiles, 32 on the others."""
    import torch

    from paper_2209_13168_amd import ecmd

    sen, tau = ecmd.sensor(640, 480, (320.0, 240.0)), 0.25
    arrs = (*_crossing(n), np.array([0, n], np.int64), np.array([tau], np.float32))
    with ecmd.Context(0) as ctx:
        want = ctx.estimate_batched(sen, *arrs, 0.0, 1.5, 1e-4)
        out = ecmd.BatchPlan.result_buffer(1)
        ctx.estimate_batched_noalloc(sen, *(torch.from_numpy(v).cuda() for v in arrs), 0.0, 1.5, 1e-4, n, out)
        torch.cuda.synchronize()
        assert ecmd.BatchPlan.results(out, 1) == want
