"""Memory that runs out: what a call can do without (the lists of the node
groups, the pixels sorted for the hot-pixel filter) is cut or left out instead
of the call being refused, and the lists are given back when another buffer
needs the room."""

import ctypes as C

import numpy as np
import pytest

from tests import host_runtime

MIB = 1 << 20
B = 8
EPS = 1e-4


@pytest.fixture(scope="module")
def so(tmp_path_factory):
    return host_runtime.build(tmp_path_factory.mktemp("rt"))


def _search(rt, ctx, n=64, windows=B):
    from paper_2209_13168_amd import ecmd

    rt.rt_windows(windows)
    x = np.zeros(n, np.float32)
    off = np.linspace(0, n, windows + 1).astype(np.int64)
    tau = np.full(windows, 0.25, np.float32)
    r = ctx.estimate_batched(ecmd.sensor(346, 260, (173, 130)), x, x, x, off, tau, 0.0, 1.0, EPS)
    assert len(r) == windows and all(q.status == 0 for q in r)
    assert rt.rt_last() == 0  # nothing is left for the caller's next check


def _needed(rt, make):
    """Bytes that `make` cannot do without: what it takes without the lists
    (128 MiB of 1024-thread workgroups' on 256 CUs)."""
    rt.rt_peak(1)
    at = rt.rt_used()
    thing = make()
    got = rt.rt_used() - at
    assert got > 128 * MIB
    thing.close()
    return got - 128 * MIB


def searches(rt, spare):
    from paper_2209_13168_amd import ecmd

    def once():
        ctx = ecmd.Context(0, stream=0)
        _search(rt, ctx)
        return ctx

    need = _needed(rt, once)
    rt.rt_limit(rt.rt_used() + need + spare)
    ctx = once()
    _search(rt, ctx)
    # the longest lists that fit
    cap = next((c for c in (1024, 512, 256, 128, 64) if c * MIB // 8 <= spare), 0)
    assert rt.rt_used() == need + cap * MIB // 8
    ctx.close()
    assert rt.rt_used() == 0


def given_back(rt):
    """A call whose own buffers fit only where the lists were."""
    from paper_2209_13168_amd import ecmd

    ctx = ecmd.Context(0, stream=0)
    _search(rt, ctx)
    rt.rt_limit(rt.rt_used() + MIB)
    n = 2 << 20  # 8 MiB an array
    _search(rt, ctx, n)
    x = np.zeros(n, np.float32)
    ctx.resample(ecmd.sensor(346, 260, (173, 130)), ecmd.sensor(43, 32, (21, 16)), x, x, x,
                 np.array([0, 0], np.int64), 0.5, 1)
    _search(rt, ctx)
    # without the lists there is room for one that needs more, not for two
    with pytest.raises(ecmd.EcmdError) as e:
        _search(rt, ctx, 64 << 20)
    assert e.value.code == ecmd.ENOMEM and rt.rt_last() == 0
    _search(rt, ctx)


def plans(rt, spare):
    from paper_2209_13168_amd import ecmd

    ctx = ecmd.Context(0, stream=0)
    sen = ecmd.sensor(346, 260, (173, 130))
    make = lambda: ctx.batch_plan(sen, 0.0, 1.0, EPS, B, 1000)
    need = _needed(rt, make)
    base = rt.rt_used()
    rt.rt_limit(base + need + spare)
    p = make()
    cap = next((c for c in (1024, 512, 256, 128, 64) if c * MIB // 8 <= spare), 0)
    assert rt.rt_used() - base == need + cap * MIB // 8 and rt.rt_last() == 0
    a = np.zeros(64, np.float32)
    n0 = rt.rt_launches()
    assert ecmd.lib().ecmd_plan_launch(p.h, *[a.ctypes.data] * 3, None, a.ctypes.data, a.ctypes.data, B, None,
                                       a.ctypes.data) == 0
    L = ecmd.plan(sen, 0.0, 1.0, EPS)["L"]
    assert rt.rt_launches() - n0 == 8 + 4 * p.limits["max_steps"] + (L + 8 if cap else 0)
    p.close()
    rt.rt_limit(base + need - MIB)
    with pytest.raises(ecmd.EcmdError) as e:
        make()
    assert e.value.code == ecmd.ENOMEM and rt.rt_used() == base


def hot_pixels(rt, spare, launches):
    from paper_2209_13168_amd import ecmd

    ctx = ecmd.Context(0, stream=0)
    sen = ecmd.sensor(346, 260, (173, 130))
    n = 4 << 20
    x, off = np.zeros(n, np.float32), np.array([0, n], np.int64)
    ctx.resample(sen, sen, x, x, x, off, 0.5, 1)  # every buffer but the pixels' own
    rt.rt_limit(rt.rt_used() + spare)
    n0 = rt.rt_launches()
    ctx.hot_pixel_filter(sen, x, x, x, off, 3)
    assert rt.rt_launches() - n0 == launches and rt.rt_last() == 0


SPARE = [200 * MIB, 128 * MIB, 127 * MIB, 9 * MIB, 8 * MIB, 7 * MIB, 0]


@pytest.mark.parametrize("spare", SPARE)
def test_a_search_takes_the_lists_that_fit(so, spare):
    host_runtime.run(so, __name__, "searches", spare)


@pytest.mark.parametrize("spare", SPARE)
def test_a_plan_takes_the_lists_that_fit(so, spare):
    host_runtime.run(so, __name__, "plans", spare)


@pytest.mark.parametrize("spare,launches", [(16 * MIB, 8), (2 * MIB, 5)])
def test_hot_pixels_without_the_sort(so, spare, launches):
    """The sorted pixels take 2 bytes an event, the counters in memory 4 a pixel."""
    host_runtime.run(so, __name__, "hot_pixels", spare, launches)


def test_lists_make_room(so):
    host_runtime.run(so, __name__, "given_back")


def coarse_plan(rt):
    """A plan of one large window: finer tiles where there is room, else the
    ones that take a third of the records."""
    from paper_2209_13168_amd import ecmd

    ctx = ecmd.Context(0, stream=0)
    sen, n = ecmd.sensor(640, 480, (320, 240)), 1_000_000
    p = ctx.batch_plan(sen, 0.0, 1.5, EPS, 1, n)
    assert p.limits["max_records"] == 6 * n
    p.close()
    rt.rt_limit(rt.rt_used() + 60 * MIB)
    p = ctx.batch_plan(sen, 0.0, 1.5, EPS, 1, n)
    assert p.limits["max_records"] == 2 * n and rt.rt_last() == 0
    p.close()


def test_a_plan_takes_the_tiles_that_fit(so):
    host_runtime.run(so, __name__, "coarse_plan")
