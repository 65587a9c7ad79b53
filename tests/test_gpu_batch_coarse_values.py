"""Coarsest products of the staged batch by their values: the first iterate x_1 =
alpha V f of every item (one to five load cases per system, 54 to 1,728 free DOFs on
the coarsest level) against that of a solve of its system by itself, whose coarsest
product is another kernel."""
import numpy as np
import pytest

import workloads
from tests.gpu_util import np64, t64

pytestmark = pytest.mark.gpu

DIMS = [(4, 4, 4), (8, 8, 8), (12, 12, 6), (16, 12, 10), (18, 14, 14)]


@pytest.mark.parametrize("loads", [(1, 2, 3, 4, 5), (4, 1, 5, 3, 2)])
def test_first_iterates_are_those_of_single_solves(loads):
    from paper_2604_26441_amd import simpgmg
    opts = [simpgmg.default_options(*d, n_levels=2, fine_prec="f32") for d in DIMS]
    rhos = [t64(workloads.grf_rho(d, 7 + k, corr_len=2.0)) for k, d in enumerate(DIMS)]
    rng = np.random.default_rng(3)
    items = [s for s, k in enumerate(loads) for _ in range(k)]
    fs = [t64(workloads.random_face_load(DIMS[s], rng)) for s in items]
    us = [t64(np.zeros(f.numel())) for f in fs]
    b = simpgmg.setup_batch(opts, rhos)
    simpgmg.pcg_solve_batch(b, items, fs, us, rtol=1e-12, maxit=1, staged=True)
    for i, s in enumerate(items):
        u = t64(np.zeros(fs[i].numel()))
        simpgmg.pcg_solve(simpgmg.setup_hierarchy(opts[s], rhos[s]), fs[i], u, rtol=1e-12, maxit=1)
        # the same cycle with FP32 smoothing on the fine level: a few FP32 units
        # (6e-8) between the kernels, amplified by a handful of operations
        assert np.linalg.norm(np64(us[i]) - np64(u)) <= 2e-6 * np.linalg.norm(np64(u)), i
