"""The network's convolutions and weight gradients at volumes around the tiles
of their kernels (16 x 4 x 4 output voxels; runs of tiles in the weight
gradient): single voxels at the coarsest level, partial tiles on every axis,
several samples, and a volume whose weight-gradient runs hold several tiles.
Reference: the FP64 oracle with the same BF16-rounded weights."""
import numpy as np
import pytest

from oracle import bf16, unet
from tests.gpu_util import np64, t32

pytestmark = pytest.mark.gpu

VOLUMES = [(1, 8, 8, 8), (3, 8, 24, 16), (1, 40, 16, 24), (2, 16, 48, 40)]


def _net(seed):
    from paper_2604_26441_amd import simpgmg
    params = [(bf16.round_bf16(w), np.random.default_rng(seed).standard_normal(b.shape) * 0.05)
              for w, b in unet.init_params(seed=seed)]
    net = simpgmg.UNet(seed=1)
    net.set_params(np.concatenate([np.concatenate([w.ravel(), b.ravel()]) for w, b in params]))
    return net, params


@pytest.mark.parametrize("vol", VOLUMES)
def test_forward(vol):
    N, D, H, W = vol
    net, params = _net(3)
    x = np.random.default_rng(8).standard_normal((N, 5, D, H, W)).astype(np.float32)
    y = np64(net.forward(t32(x)))
    ref, _ = unet.forward(params, x.astype(np.float64))
    # eight FP32 sums of up to 27 * 128 exact products: 8 * sqrt(3456) * 2^-24
    # = 2.8e-5 of the largest value
    assert np.abs(y - ref).max() <= 3e-5 * np.abs(ref).max()


@pytest.mark.parametrize("vol", VOLUMES)
def test_gradients(vol):
    N, D, H, W = vol
    net, params = _net(4)
    g = np.random.default_rng(9)
    x = g.standard_normal((N, 5, D, H, W)).astype(np.float32).astype(np.float64)
    t = g.standard_normal((N, 3, D, H, W)).astype(np.float32).astype(np.float64)
    loss, grads = net.grad(t32(x), t32(t))
    y, cache = unet.forward(params, x)
    lref, dy = unet.loss_mse(y, t, np.ones((N, 1, D, H, W)))
    off = 0
    for dw, db in unet.backward(params, cache, dy):
        gw = grads[off:off + dw.size].reshape(dw.shape)
        gb = grads[off + dw.size:off + dw.size + db.size]
        off += dw.size + db.size
        # a rounding that crosses a ReLU's zero moves whole terms: the bound of
        # the smaller volume's test
        assert np.linalg.norm(gw - dw) <= 1e-3 * np.linalg.norm(dw)
        assert np.linalg.norm(gb - db) <= 1e-3 * max(np.linalg.norm(db), 1e-12)
    assert off == grads.size and abs(loss - lref) <= 1e-5 * abs(lref)
