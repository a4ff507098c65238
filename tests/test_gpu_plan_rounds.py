"""A plan's searches that outlast the rounds in which node groups are formed
equal the synchronous call's, which forms them in every round."""

import numpy as np
import pytest

from synth import config_windows, pack_batch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("F,max_steps", [(1, 400), (2, 400), (4, 200), (96, 8), (96, 60)])
def test_searches_past_the_node_rounds(F, max_steps):
    import torch

    from paper_2209_13168_amd import ecmd

    wins = config_windows("c1", range(8), n_events=6000)
    s = wins[0].spec
    arrs = pack_batch(wins)
    sen = ecmd.sensor(s.width, s.height, s.foe)
    with ecmd.Context(0) as ctx:
        want = ctx.estimate_batched(sen, *arrs, s.d_lo, s.d_hi, s.eps, frontier_batch=F)
        L = want[0].L
        if F < 4:
            assert max(r.steps for r in want) > L + 8
        plan = ctx.batch_plan(sen, s.d_lo, s.d_hi, s.eps, 8, int(arrs[3][-1]), frontier_batch=F, max_steps=max_steps)
        out = plan.result_buffer(8)
        dev = [torch.from_numpy(a).cuda() for a in arrs]
        for _ in range(2):
            out.zero_()
            plan.launch(*dev, out)
            torch.cuda.synchronize()
            got = plan.results(out, 8)
            for g, w in zip(got, want):
                if w.steps >= max_steps:
                    assert g.status == ecmd.EBUDGET and g.steps == max_steps
                else:
                    assert g == w
