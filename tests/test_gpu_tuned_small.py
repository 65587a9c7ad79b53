"""Tuned solves on small meshes, where the fastest FP64 product and the fastest one
with p.q may be different forms: in the tuned hierarchy and in the next one of the
same mesh (which takes the kept shapes) they give the untuned solve's result."""
import numpy as np
import pytest

import workloads
from tests.gpu_util import np64, t64

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dims", [(10, 7, 5), (21, 18, 13), (26, 25, 24)])
@pytest.mark.parametrize("prec", ["f64", "f32", "bf16x3"])
def test_tuned_solve_is_the_untuned_one(dims, prec):
    from paper_2604_26441_amd import simpgmg
    opts = simpgmg.default_options(*dims, n_levels=2, fine_prec=prec)
    rho = t64(np.random.default_rng(6).uniform(0.2, 1.0, np.prod(dims)))
    f = t64(workloads.edge_load(dims))

    def solve(h):
        u = t64(np.zeros(f.numel()))
        r = simpgmg.pcg_solve(h, f, u, rtol=1e-11, maxit=200)
        assert r["status"] == "converged" and r["rel_res_true"] < 1e-11
        return r["iters"], np64(u)

    h = simpgmg.setup_hierarchy(opts, rho)
    for rows, planes in ((1, 4), (0, 0), (4, 2)):
        simpgmg.set_launch_shape(h, "f64", rows, planes)
        it, want = solve(h)
    simpgmg.autotune(h)
    for k in (h, simpgmg.setup_hierarchy(opts, rho)):
        n, got = solve(k)
        assert abs(n - it) <= 1
        # residuals of 1e-11 on both sides, and a condition number below 1e4 at
        # these contrasts and sizes
        assert np.linalg.norm(got - want) <= 1e-7 * np.linalg.norm(want)
