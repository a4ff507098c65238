"""The network's input at the lines between its chunk sizes (windows of fewer
than 2048 events on the mean; 8 million events in the call) and at the chunks'
edges, bit for bit."""

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("sizes", [
    [2048, 2047, 2048], [2048, 2048, 2048],              # either side of the mean
    [0, 4095, 0, 4096, 4097] + [1] * 40,                 # small chunks
    [8191, 8192, 8193, 0, 70_001],                       # middle ones
    [7_999_999], [5_000_000, 0, 3_000_000],              # either side of the total
], ids=lambda s: "-".join(map(str, s[:5])))
def test_input_at_the_rules_edges(sizes):
    import torch

    from paper_2209_13168_amd import ecmd

    W, H = 346, 260
    r = np.random.default_rng(len(sizes))
    n = sum(sizes)
    x, y = (r.random(n).astype(np.float32) * np.float32(s) for s in (W, H))
    off = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int64)
    bx = np.clip(np.floor(x * np.float32(64) / np.float32(W)), 0, 63).astype(np.int64)
    by = np.clip(np.floor(y * np.float32(64) / np.float32(H)), 0, 63).astype(np.int64)
    want = []
    for a, b in zip(off, off[1:]):
        cnt = np.bincount(by[a:b] * 64 + bx[a:b], minlength=4096).astype(np.float32)
        u = (cnt * (np.float32(4096) / np.float32(b - a) if b > a else np.float32(0))).astype(np.float32).view(np.uint32)
        want.append(((u + 0x7FFF + ((u >> 16) & 1)) >> 16).astype(np.uint16))
    with ecmd.Context(0) as ctx:
        sen = ecmd.sensor(W, H, (W / 2, H / 2))
        got = ctx.downsample(sen, x, y, off)
        dev = ctx.downsample(sen, *(torch.from_numpy(a).cuda() for a in (x, y, off)))
    assert np.array_equal(got.reshape(len(sizes), 4096), want)
    assert np.array_equal(dev.cpu().numpy().reshape(len(sizes), 4096), want)
