"""Preprocessing of many small windows: chunks that hold several windows,
more bands than one workgroup each takes, more windows than a grid holds
workgroups; against the CPU statement, bit for bit."""

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

# small windows between large ones, at the edges of chunks (8192 events) and
# keep words; many windows a chunk; empty ones first, last and between
SIZES = {
    "mixed": [0, 20_000] + [1] * 300 + [0] * 50 + [9000] + [3] * 5000 + [8192, 8191, 1, 0],
    "small": [0, 0] + [63, 64, 65, 0, 1, 2] * 400,
    "two": [8191, 8194],
    "bands": [7] * 10_000 + [5000] + [2, 0, 9] * 2500,  # 17501 windows, more than 16384 bands
}


@pytest.fixture(scope="module")
def ctx():
    from paper_2209_13168_amd import ecmd

    c = ecmd.Context(0)
    yield c
    c.close()


def _events(sizes, W, H, seed):
    """Events on few enough pixels that some hold several, some off the sensor."""
    r = np.random.default_rng(seed)
    n = int(np.sum(sizes))
    px = np.unique(np.concatenate([[0, W * H - 1], r.integers(0, W * H, 300)]))
    pix = px[r.integers(0, 12, n) * (px.size // 12)]
    x = (pix % W + r.random(n)).astype(np.float32)
    y = (pix // W + r.random(n)).astype(np.float32)
    off_sensor = r.random(n) < 0.02
    x[off_sensor] = r.choice(np.array([-0.5, W, W + 3.0, -1e9], np.float32), int(off_sensor.sum()))
    off = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int64)
    return x, y, r.random(n).astype(np.float32), off


def _check(got, want, what):
    for g, w in zip(got, want):
        assert np.array_equal(g if isinstance(g, np.ndarray) else g.cpu().numpy(), w), what


@pytest.mark.parametrize("W,H", [(1, 1), (128, 128), (129, 128), (346, 260), (2100, 2000)])
@pytest.mark.parametrize("sizes", SIZES)
def test_hot_pixels(ctx, W, H, sizes):
    import torch

    from oracle import preproc
    from paper_2209_13168_amd import ecmd

    n = SIZES[sizes]
    if W > 1000:  # counters in memory, 17 MB a window
        n = n[:400]
    x, y, t, off = _events(n, W, H, 3)
    sen = ecmd.sensor(W, H, (W / 2, H / 2))
    first = 5 if off[-1] > 20 else 0  # device arrays whose windows start later
    dev = [torch.from_numpy(np.concatenate([np.full(first, 0.25, np.float32), a])).cuda() for a in (x, y, t)]
    for most in (0, 2, 400):
        # (the oracle, but counted over all windows at once)
        win = np.repeat(np.arange(len(n)), n)
        ins = (x >= 0) & (x < W)
        key, inv, cnt = np.unique(win[ins] * (W * H) + np.floor(y[ins]).astype(np.int64) * W +
                                  np.floor(x[ins]).astype(np.int64), return_inverse=True, return_counts=True)
        keep = np.ones(x.size, bool)
        keep[ins] = cnt[inv] <= most
        want = preproc._compact(x, y, t, off, keep)
        if len(n) < 1000:
            _check(preproc.hot_pixel_filter(x, y, t, off, W, H, most), want, "the two statements")
        _check(ctx.hot_pixel_filter(sen, x, y, t, off, most), want, (W, H, sizes, most))
        _check(ctx.hot_pixel_filter(sen, *dev, torch.from_numpy(off + first).cuda(), most), want,
               (W, H, sizes, most, "device"))


@pytest.mark.parametrize("sizes", SIZES)
def test_resample(ctx, sizes):
    from oracle import preproc
    from paper_2209_13168_amd import ecmd

    x, y, t, off = _events(SIZES[sizes], 346, 260, 4)
    got = ctx.resample(ecmd.sensor(346, 260, (173, 130)), ecmd.sensor(43, 32, (21, 16)), x, y, t, off, 0.25, 77)
    _check(got, preproc.resample(x, y, t, off, 346, 260, 43, 32, 0.25, 77), sizes)


def test_more_windows_than_workgroups_in_a_grid(ctx):
    """4.3 million windows of an event or two on a 2 x 2 sensor: a workgroup of
    1024 threads per window would exceed the 2^32 threads of a launch."""
    import torch

    from oracle import preproc
    from paper_2209_13168_amd import ecmd

    B = 4_300_000
    r = np.random.default_rng(8)
    n = r.integers(1, 3, B)
    off = np.concatenate([[0], np.cumsum(n)]).astype(np.int64)
    N = int(off[-1])
    x, y, t = (r.random(N).astype(np.float32) * np.float32(s) for s in (2.0, 2.0, 1.0))
    dev = [torch.from_numpy(a).cuda() for a in (x, y, t, off)]
    win = np.repeat(np.arange(B), n)
    pix = win * 4 + np.floor(y).astype(np.int64) * 2 + np.floor(x).astype(np.int64)
    z = (win.astype(np.uint64) << np.uint64(32)) + (np.arange(N) - off[win]).astype(np.uint64) + np.uint64(1)
    with np.errstate(over="ignore"):
        draw = preproc._mix(np.uint64(77) + z * preproc.GOLDEN) >> np.uint64(40)
    sen, small = ecmd.sensor(2, 2, (1, 1)), ecmd.sensor(1, 1, (0.5, 0.5))
    for keep, got, sc in ((np.bincount(pix, minlength=4 * B)[pix] <= 1, ctx.hot_pixel_filter(sen, *dev, 1), 1.0),
                          (draw < np.uint64(1 << 22), ctx.resample(sen, small, *dev, 0.25, 77), 0.5)):
        sc = np.float32(sc)
        want = (x[keep] * sc, y[keep] * sc, t[keep], np.concatenate([[0], np.cumsum(keep)])[off])
        _check(got, want, float(sc))
