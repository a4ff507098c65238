"""Windows of one batch take their steps at their own pace: a window whose
endpoint certificates fail needs a second round for the step, the others do
not wait for it.  Batches that mix both kinds, cut at several step limits,
return for every window what that window returns alone."""

import dataclasses

import numpy as np
import pytest

from synth import config_windows, pack_batch
from synth.ventral import make_window

pytestmark = pytest.mark.gpu


def _still(base, n):
    """n events at the FOE: they never move, so every right child's
    certificate fails."""
    s = base.spec
    w = make_window(dataclasses.replace(s, n_events=0), 1, 7)
    return dataclasses.replace(w, x=np.full(n, s.foe[0], np.float32), y=np.full(n, s.foe[1], np.float32),
                               t_rel=np.linspace(0, 0.4, n).astype(np.float32), p=np.ones(n, np.int8),
                               owner=np.full(n, -1, np.int32))


@pytest.mark.parametrize("max_steps", [4, 8, 0])
def test_mixed_batch_equals_its_windows_alone(max_steps):
    import torch

    from paper_2209_13168_amd import ecmd

    base = config_windows("c1", [0, 1])
    s = base[0].spec
    wins = [_still(base[0], 5), base[0], _still(base[0], 1), base[1]]
    sen = ecmd.sensor(s.width, s.height, s.foe)
    with ecmd.Context(0) as ctx:
        plan = ctx.batch_plan(sen, s.d_lo, s.d_hi, s.eps, max_windows=4, max_events=100_000, max_steps=max_steps)

        def launch(ws):
            args = [torch.from_numpy(a).cuda() for a in pack_batch(ws)]
            out = plan.result_buffer(len(ws))
            plan.launch(*args, out)
            torch.cuda.synchronize()
            return plan.results(out, len(ws))

        got = launch(wins)
        alone = [launch([w])[0] for w in wins]
        plan.close()
        assert got == alone
        assert got[0].bound_evals > 0 and got[0].bound_certs > 0
        if max_steps:
            assert [r.status for r in got] == [ecmd.EBUDGET] * 4 and {r.steps for r in got} == {max_steps}
        else:
            x, y, t, off, tau = pack_batch(wins)
            assert got == ctx.estimate_batched(sen, x, y, t, off, tau, s.d_lo, s.d_hi, s.eps)
