"""Coarsest products of the staged batch from the triangle's tiles: 54, 300, 504,
1008 and 1728 free DOFs (one tile; a partial strip; exactly one strip of eight
tiles; two; 27 whole tiles), one to five load cases each, against a solve of
each system by itself."""
import numpy as np
import pytest

import workloads
from tests.gpu_util import t64

pytestmark = pytest.mark.gpu

DIMS = [(4, 4, 4), (8, 8, 8), (12, 12, 6), (16, 12, 10), (18, 14, 14)]


@pytest.mark.parametrize("loads", [(1, 2, 3, 4, 5), (4, 1, 5, 3, 2)])
def test_items_match_the_single_solves(loads):
    import torch
    from paper_2604_26441_amd import simpgmg
    opts = [simpgmg.default_options(*d, n_levels=2, fine_prec="bf16x3") for d in DIMS]
    rhos = [t64(workloads.grf_rho(d, 7 + k, corr_len=2.0)) for k, d in enumerate(DIMS)]
    rng = np.random.default_rng(3)
    items = [s for s, k in enumerate(loads) for _ in range(k)]
    fs = [t64(workloads.random_face_load(DIMS[s], rng)) for s in items]
    us = [torch.zeros_like(f) for f in fs]
    b = simpgmg.setup_batch(opts, rhos)
    res, _ = simpgmg.pcg_solve_batch(b, items, fs, us, rtol=1e-9, maxit=300, staged=True)
    for i, s in enumerate(items):
        h = simpgmg.setup_hierarchy(opts[s], rhos[s])
        u = torch.zeros_like(fs[i])
        one = simpgmg.pcg_solve(h, fs[i], u, rtol=1e-9, maxit=300)
        assert res[i]["status"] == one["status"] == "converged"
        # both residuals are below 1e-9 of the load; the error is at most cond(K)
        # (<= 1e4 with these contrasts) times that, and close to it only if the
        # two iterations had nothing in common
        assert float((u - us[i]).norm()) <= 1e-6 * float(u.norm())
        assert abs(res[i]["iters"] - one["iters"]) <= 1
