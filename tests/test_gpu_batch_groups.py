"""Coarsest solves of the staged batch shared between the load cases of a
system: one, four (one full group) and six (two groups) load cases of three
systems, the coarsest sizes not multiples of the row block.  Each item must
have the result it has when its system's other load cases are not there."""
import numpy as np
import pytest

import workloads
from tests.gpu_util import t64

pytestmark = pytest.mark.gpu


def test_shared_pass_gives_each_item_its_own_result():
    import torch
    from paper_2604_26441_amd import simpgmg
    dims = [(12, 6, 6), (10, 9, 7), (16, 8, 8)]
    loads = [1, 4, 6]
    opts = [simpgmg.default_options(*d, n_levels=2, fine_prec="bf16x3") for d in dims]
    rhos = [t64(workloads.grf_rho(d, 40 + k, corr_len=2.0)) for k, d in enumerate(dims)]
    rng = np.random.default_rng(5)
    items = [s for s, k in enumerate(loads) for _ in range(k)]
    fs = [t64(workloads.random_face_load(dims[s], rng)) for s in items]
    b = simpgmg.setup_batch(opts, rhos)
    us = [torch.zeros_like(f) for f in fs]
    res, _ = simpgmg.pcg_solve_batch(b, items, fs, us, rtol=1e-8, maxit=300, staged=True)
    assert all(r["status"] == "converged" for r in res)
    for i, s in enumerate(items):
        u = torch.zeros_like(fs[i])
        (r,), _ = simpgmg.pcg_solve_batch(b, [s], [fs[i]], [u], rtol=1e-8, maxit=300, staged=True)
        assert r["iters"] == res[i]["iters"]
        # the item set's launch shapes are timed and may differ between the two
        # calls, which moves the FP64 operator's rounding: 1e-16 of K u through
        # a solve to 1e-8
        assert float((u - us[i]).norm()) <= 1e-9 * float(us[i].norm())
