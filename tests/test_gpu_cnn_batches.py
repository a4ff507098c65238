"""Training batches of the network at the sizes where the batch sum changes
its split over waves, and images whose events lie on the borders of the
planes (the zero rows and columns that the taps read)."""

import numpy as np
import pytest

from tests.test_oracle_cnn import _rand

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    from paper_2209_13168_amd import ecmd

    c = ecmd.Context(0)
    yield c
    c.close()


@pytest.mark.parametrize("B", [1, 2, 4, 8, 16, 64])
def test_batch_gradient_is_the_mean_of_its_images(ctx, B):
    """B a power of two: 1/B scales every image's gradient exactly, so only
    the sum over the images rounds: B additions, half an ulp of a partial sum
    (at most the sum of magnitudes) each."""
    from paper_2209_13168_amd import ecmd

    net = ecmd.Cnn(ctx, seed=4)
    p, x, y = _rand(11, B=B)
    net.set_params(p)
    imgs = x.reshape(B, -1)
    g, loss = net.grads(imgs, y)
    one = [net.grads(imgs[k:k + 1], y[k:k + 1]) for k in range(B)]
    each = np.array([v[0] for v in one], np.float64) / B
    tol = B * 2.0**-24 * np.abs(each).sum(0)
    assert (np.abs(g - each.sum(0)) <= tol).all()
    losses = np.array([v[1] for v in one], np.float64) / B
    assert abs(loss - losses.sum()) <= (B + 2) * 2.0**-24 * losses.sum()
    assert np.array_equal(net.forward(imgs), np.concatenate([net.forward(imgs[k:k + 1]) for k in range(B)]))
    net.close()


@pytest.mark.parametrize("name,ys,xs", [("corners", [0, 0, 63, 63], [0, 63, 0, 63]), ("top", [0] * 64, range(64)),
                                        ("right", range(64), [63] * 64), ("bottom", [63] * 64, range(64)),
                                        ("empty", [], [])])
def test_border_images(ctx, name, ys, xs):
    """Against the fp64 statement, with the bounds of
    tests/test_gpu_cnn.py: |g - g64| <= 2^-7 |g64| + 2^-9 max|g64| per layer."""
    from oracle import cnn as ocnn
    from paper_2209_13168_amd import ecmd

    net = ecmd.Cnn(ctx, seed=4)
    p, _, _ = _rand(3, B=1)
    img = np.zeros((1, 64, 64), np.float32)
    img[0, list(ys), list(xs)] = 1.0 + 0.5 * (np.arange(len(ys)) % 3)
    bits = (img.view(np.uint32) >> 16).astype(np.uint16)  # exact in bfloat16
    y = np.array([0.3], np.float32)
    net.set_params(p)
    g, loss = net.grads(bits.reshape(1, -1), y)
    loss_o, g_o, _ = ocnn.loss_and_grad(p, bits, y, rounding=True)
    assert loss == pytest.approx(loss_o, rel=1e-2)
    k = 0
    for layer, shape in ocnn.SHAPES:
        n = int(np.prod(shape))
        a, b = g[k:k + n].astype(np.float64), g_o[k:k + n]
        assert (np.abs(a - b) <= 2.0**-7 * np.abs(b) + 2.0**-9 * np.abs(b).max()).all(), (name, layer)
        k += n
    net.close()
