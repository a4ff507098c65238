"""The captured rounds of the graph tuning are kept while nothing that they
depend on changes: equal searches capture once."""

import numpy as np
import pytest

from tests import host_runtime


@pytest.fixture(scope="module")
def so(tmp_path_factory):
    return host_runtime.build(tmp_path_factory.mktemp("rt"))


def equal_searches(rt):
    from paper_2209_13168_amd import ecmd

    ctx = ecmd.Context(0, stream=0)
    ctx.set_tuning(graph=True)
    B, n = 8, 64
    rt.rt_windows(B)
    x = np.zeros(n, np.float32)
    off = np.linspace(0, n, B + 1).astype(np.int64)
    tau = np.full(B, 0.25, np.float32)
    sen = ecmd.sensor(346, 260, (173, 130))

    def search(eps=1e-4):
        ctx.estimate_batched(sen, x, x, x, off, tau, 0.0, 1.0, eps)

    search()
    assert rt.rt_instantiated() == 1
    rng = np.random.default_rng(2)
    for k in range(40):
        # other calls leave other values on the stack
        for _ in range(int(rng.integers(0, 4))):
            ecmd.plan(ecmd.sensor(int(rng.integers(1, 1500)), int(rng.integers(1, 900)), rng.uniform(0, 900, 2)), 0.0,
                      float(rng.uniform(0.1, 2)), float(rng.uniform(1e-6, 1e-2)))
            ctx.probe_point(sen, x, x, x, 0.25, rng.uniform(0, 1, int(rng.integers(1, 9))).astype(np.float32))
        if k % 3 == 0:
            ctx.hot_pixel_filter(sen, x, x, x, off, int(rng.integers(0, 99)))
        rt.rt_scribble(int(rng.integers(0, 256)))
        search()
    assert rt.rt_instantiated() == 1
    search(1e-5)
    assert rt.rt_instantiated() == 2


def test_equal_searches_capture_once(so):
    host_runtime.run(so, __name__, "equal_searches")
