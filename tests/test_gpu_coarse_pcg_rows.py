"""Coarsest PCG on grids whose 64-node blocks fill the chip about once, where a block
does all three rows: with the neighbours staged in LDS and on a grid too long for
that.  Reference: the oracle's V-cycle."""
import numpy as np
import pytest

import workloads
from oracle import mesh, multigrid
from tests.gpu_util import np64, rel_err, t64

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dims", [(140, 138, 2), (280, 70, 2)])
def test_vcycle_matches_the_oracle(dims):
    from paper_2604_26441_amd import simpgmg
    rho = np.random.default_rng(5).uniform(0.1, 1.0, np.prod(dims))
    fixed = workloads.cantilever_fixed(dims).astype(bool)
    oh = multigrid.build(dims, mesh.simp_modulus(rho, 3), fixed, multigrid.Options(
        n_levels=2, dense_max=10, coarse_pcg_iters=3, lambdas=[2.0]))
    o = simpgmg.default_options(*dims, n_levels=2, fine_prec="f64", dense_max=10, coarse_pcg_iters=3)
    h = simpgmg.setup_hierarchy(o, t64(rho), lambda_override=[2.0])
    r = workloads.random_vector(fixed.size, 6, fixed)
    z = t64(np.zeros_like(r))
    simpgmg.vcycle(h, t64(r), z)
    # three steps: no drift beyond rounding
    assert rel_err(np64(z), multigrid.vcycle(oh, r), np64(z)) < 1e-11
