"""Concurrent batch solve with worker threads on systems on both sides of 100,000
DOFs, two load cases each: the workers replay the systems' iteration graphs, so
every item is bitwise the solve of its system by itself, by one worker or by
three, also where the systems were set up without graphs."""
import numpy as np
import pytest

import workloads
from tests.gpu_util import np64, t64

pytestmark = pytest.mark.gpu

DIMS = [(34, 32, 32), (16, 12, 12), (30, 34, 33), (33, 33, 30)]


@pytest.mark.parametrize("workers,use_graphs", [(1, 1), (3, 1), (3, 0)])
def test_items_are_the_single_solves(workers, use_graphs):
    from paper_2604_26441_amd import simpgmg
    opts = [simpgmg.default_options(*d, n_levels=3, fine_prec="bf16x3", use_graphs=use_graphs)
            for d in DIMS]
    rhos = [t64(workloads.grf_rho(d, 11 + k)) for k, d in enumerate(DIMS)]
    rng = np.random.default_rng(4)
    items = [s for s in range(len(DIMS)) for _ in range(2)]
    fs = [t64(workloads.random_face_load(DIMS[s], rng)) for s in items]
    us = [t64(np.zeros(f.numel())) for f in fs]
    b = simpgmg.setup_batch(opts, rhos)
    res, _ = simpgmg.pcg_solve_batch_concurrent(b, items, fs, us, rtol=1e-8, maxit=200, workers=workers)
    for i, s in enumerate(items):
        u = t64(np.zeros(fs[i].numel()))
        one = simpgmg.pcg_solve(simpgmg.setup_hierarchy(opts[s], rhos[s]), fs[i], u, rtol=1e-8, maxit=200)
        assert (res[i]["status"], res[i]["iters"]) == (one["status"], one["iters"]) and one["status"] == "converged"
        assert np.array_equal(np64(us[i]), np64(u))
