"""What a plan's launch enqueues, counted on the host."""

import numpy as np
import pytest

from tests import host_runtime


@pytest.fixture(scope="module")
def so(tmp_path_factory):
    return host_runtime.build(tmp_path_factory.mktemp("rt"))


def plan_launches(rt, max_steps, groups):
    import ctypes as C

    from paper_2209_13168_amd import ecmd

    ctx = ecmd.Context(0, stream=0)
    sen = ecmd.sensor(346, 260, (173, 130))
    eps = 1e-4
    L = ecmd.plan(sen, 0.0, 1.0, eps)["L"]
    B = 8 if groups else 1
    p = ctx.batch_plan(sen, 0.0, 1.0, eps, B, 100_000, max_steps=max_steps)
    a = np.zeros(64, np.float32)
    n0 = rt.rt_launches()
    rc = ecmd.lib().ecmd_plan_launch(p.h, *[a.ctypes.data] * 3, None, a.ctypes.data, a.ctypes.data, B, None,
                                     a.ctypes.data)
    n = rt.rt_launches() - n0
    assert rc == 0
    # check, window parameters, clear, count, scan, scatter, first hypotheses,
    # results; a step's two evaluations and frontiers; the groups' launches
    assert n == 8 + 4 * max_steps + (L + 8 if groups else 0), (n, max_steps, L)


@pytest.mark.parametrize("max_steps", [36, 200])
@pytest.mark.parametrize("groups", [False, True])
def test_a_plan_launches_node_groups_in_its_first_rounds(so, max_steps, groups):
    """A round's launches cost their time empty or not: those of the node
    groups come on top of a step's four in the first L + 8 rounds only."""
    host_runtime.run(so, __name__, "plan_launches", max_steps, groups)
