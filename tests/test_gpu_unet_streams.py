"""First calls of the network on a stream of their own while the default stream is
busy: the buffers that these calls allocate are cleared in their own order, so the
results are those of the same calls on the default stream."""
import numpy as np
import pytest

from tests.gpu_util import np64, t32

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("what", ["params", "forward", "gradients"])
def test_first_call_on_a_side_stream(what):
    import torch
    from paper_2604_26441_amd import simpgmg
    g = np.random.default_rng(2)
    x, t = t32(g.standard_normal((1, 5, 24, 16, 16))), t32(g.standard_normal((1, 3, 24, 16, 16)))
    big = torch.zeros(1 << 28, device="cuda:0")

    def call(stream):
        net = simpgmg.UNet(seed=3)
        torch.cuda.synchronize()
        if stream is not None:
            for _ in range(8):
                big.add_(1.0)                   # the default stream's own work
        if what == "params":
            return net.get_params(stream=stream)
        if what == "forward":
            y = net.forward(x, stream=stream)
            torch.cuda.synchronize()
            return np64(y)
        return net.grad(x, t, stream=stream)[1]

    want = call(None)
    side = torch.cuda.Stream()
    for _ in range(3):
        assert np.array_equal(call(side), want)
