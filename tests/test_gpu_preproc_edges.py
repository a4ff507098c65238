"""Preprocessing at the edges of its chunks, keep words and pixel bands,
against the CPU statement, bit for bit."""

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

# windows around the chunk (8192) and the keep word (64), empty ones between
SIZES = [[0], [1], [63, 64, 65], [0, 8191, 0, 8192, 8193, 0], [0, 0, 9000, 1, 0, 24_577]]
# one pixel; exactly one band of 16384 pixels; one pixel row more; several
# bands with a ragged end; more bands than the sort takes (counters in memory)
SENSORS = [(1, 1), (128, 128), (129, 128), (346, 260), (2100, 2000)]


@pytest.fixture(scope="module")
def ctx():
    from paper_2209_13168_amd import ecmd

    c = ecmd.Context(0)
    yield c
    c.close()


def _events(sizes, W, H, seed):
    """Events on few enough pixels that some hold several, some off the sensor."""
    r = np.random.default_rng(seed)
    n = sum(sizes)
    k = r.integers(0, 400, n)
    px = np.unique(np.concatenate([[0, W * H - 1], r.integers(0, W * H, 300)]))
    pix = px[k % px.size]
    x = (pix % W + r.random(n)).astype(np.float32)
    y = (pix // W + r.random(n)).astype(np.float32)
    off_sensor = r.random(n) < 0.02
    x[off_sensor] = r.choice(np.array([-0.5, W, W + 3.0, -1e9], np.float32), int(off_sensor.sum()))
    off = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int64)
    return x, y, r.random(n).astype(np.float32), off


@pytest.mark.parametrize("W,H", SENSORS)
@pytest.mark.parametrize("sizes", SIZES, ids=["-".join(map(str, s)) for s in SIZES])
def test_hot_pixels(ctx, W, H, sizes):
    import torch

    from oracle import preproc
    from paper_2209_13168_amd import ecmd

    x, y, t, off = _events(sizes, W, H, 3)
    sen = ecmd.sensor(W, H, (W / 2, H / 2))
    for most in (0, 1, 12):
        want = preproc.hot_pixel_filter(x, y, t, off, W, H, most)
        got = ctx.hot_pixel_filter(sen, x, y, t, off, most)
        dev = ctx.hot_pixel_filter(sen, *(torch.from_numpy(a).cuda() for a in (x, y, t, off)), most)
        for g, d, w in zip(got, dev, want):
            assert np.array_equal(g, w) and np.array_equal(d.cpu().numpy(), w), (W, H, sizes, most)


@pytest.mark.parametrize("sizes", SIZES, ids=["-".join(map(str, s)) for s in SIZES])
@pytest.mark.parametrize("keep", [0.0, 0.25, 1.0])
def test_resample(ctx, sizes, keep):
    from oracle import preproc
    from paper_2209_13168_amd import ecmd

    x, y, t, off = _events(sizes, 346, 260, 4)
    got = ctx.resample(ecmd.sensor(346, 260, (173, 130)), ecmd.sensor(43, 32, (21, 16)), x, y, t, off, keep, 77)
    want = preproc.resample(x, y, t, off, 346, 260, 43, 32, keep, 77)
    for g, w in zip(got, want):
        assert np.array_equal(g, w), (sizes, keep)


@pytest.mark.parametrize("sizes", [[0], [1, 0, 5], [32_767, 32_768, 32_769]])
def test_downsample(ctx, sizes):
    from paper_2209_13168_amd import ecmd

    x, y, _, off = _events(sizes, 346, 260, 5)
    got = ctx.downsample(ecmd.sensor(346, 260, (173, 130)), x, y, off).reshape(len(sizes), 64, 64)
    for k, n in enumerate(sizes):
        a, b = off[k], off[k + 1]
        bx = np.clip(np.floor(x[a:b] * np.float32(64) / np.float32(346)), 0, 63).astype(int)
        by = np.clip(np.floor(y[a:b] * np.float32(64) / np.float32(260)), 0, 63).astype(int)
        cnt = np.zeros((64, 64), np.float32)
        np.add.at(cnt, (by, bx), 1)
        u = (cnt * (np.float32(4096) / np.float32(max(n, 1)) if n else np.float32(0))).astype(np.float32).view(np.uint32)
        want = ((u + 0x7FFF + ((u >> 16) & 1)) >> 16).astype(np.uint16)
        assert np.array_equal(got[k], want)
