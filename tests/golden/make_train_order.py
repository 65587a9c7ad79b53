"""Writes train_order.json: per seed and parameter block (weights, then biases, of the
eight layers) four signed sums and the norm of the network's gradients on a 1 x
24^3 grid.  A ReLU's mask is a step function of the value before it, so these seeds'
gradients move by 5e-4 of their norm and more when the training forward's sums are
rounded in another order; the kept values are those of the library's first training
pass (one sum per output, terms from the smallest, decoder inputs expanded).

Usage, on a machine with the GPU: python -m tests.golden.make_train_order
"""
import json
import os

import numpy as np

PATH = os.path.join(os.path.dirname(os.path.abspath(__file__)), "train_order.json")
CHANNELS = [(5, 16, 27), (16, 32, 27), (32, 64, 27), (64, 128, 27), (128, 64, 27), (64, 32, 27), (32, 16, 27), (16, 3, 1)]
SEEDS = (13, 17, 28, 160, 215, 242)


def summary(seed):
    import torch
    from paper_2604_26441_amd import simpgmg
    off = np.cumsum([0] + [n for ci, co, taps in CHANNELS for n in (ci * co * taps, co)])
    signs = np.random.default_rng(77).integers(0, 2, (4, off[-1])) * 2.0 - 1
    g = np.random.default_rng(seed)
    x = g.standard_normal((1, 5, 24, 24, 24)).astype(np.float32)
    t = g.standard_normal((1, 3, 24, 24, 24)).astype(np.float32)
    net = simpgmg.UNet(seed=seed)
    grads = net.grad(torch.tensor(x, device="cuda:0"), torch.tensor(t, device="cuda:0"))[1].astype(np.float64)
    blocks = [slice(a, b) for a, b in zip(off[:-1], off[1:])]
    return np.array([[float((s[b] * grads[b]).sum()) for s in signs] + [float(np.linalg.norm(grads[b]))] for b in blocks])


if __name__ == "__main__":
    with open(PATH, "w") as fh:
        json.dump({str(s): summary(s).tolist() for s in SEEDS}, fh, indent=0)
