"""FGMRES basis kernels at the edges of their column groups (8 columns per pass
of the products; a row of 8, 16, 24 or 32 columns in registers, more from memory
again), and the coarsest PCG on grids of whole and partial 64-node blocks and on
one too long for its LDS bands."""
import numpy as np
import pytest

import workloads
from oracle import krylov, mesh, multigrid
from tests.gpu_util import np64, rel_err, t64

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("cols", [1, 7, 8, 9, 16, 17, 24, 25, 32, 33, 40, 63])
def test_arnoldi_over_columns_matches_the_oracle(cols):
    from paper_2604_26441_amd import simpgmg
    dims = (9, 8, 7)
    rho = np.random.default_rng(cols).uniform(0.2, 1.0, np.prod(dims))
    fixed = workloads.cantilever_fixed(dims).astype(bool)
    K = mesh.assemble(dims, mesh.simp_modulus(rho, 3), fixed=fixed)
    dinv = np.where(fixed, 0.0, 1.0 / np.maximum(K.diagonal(), 1e-300))
    f = workloads.random_vector(fixed.size, 3, fixed)
    h = simpgmg.setup_hierarchy(simpgmg.default_options(*dims, n_levels=2, fine_prec="f64"), t64(rho))
    x, _, it, ho = krylov.fgmres(lambda v: K @ v, f, lambda r: dinv * r, rtol=1e-12, maxit=cols,
                                 restart=cols)
    u = t64(np.zeros_like(f))
    res = simpgmg.fgmres_solve(h, t64(f), u, rtol=1e-12, maxit=cols, restart=cols,
                               precond=1, history_cap=80)
    assert res["iters"] == it == cols
    hg = list(res["history"])[:len(ho)]
    # two Gram-Schmidt variants: the basis differs by rounding (1e-16) times the
    # growth over at most 63 steps of a residual that falls by less than 1e6
    np.testing.assert_allclose(hg, ho, rtol=1e-6, atol=1e-13)
    assert np.linalg.norm(np64(u) - x) <= 1e-6 * np.linalg.norm(x)


@pytest.mark.parametrize("dims", [(14, 14, 6), (6, 6, 6), (13, 9, 7), (300, 4, 4)])
def test_coarsest_pcg_blocks_match_the_oracle(dims):
    from paper_2604_26441_amd import simpgmg
    rho = np.random.default_rng(5).uniform(0.1, 1.0, np.prod(dims))
    fixed = workloads.cantilever_fixed(dims).astype(bool)
    oh = multigrid.build(dims, mesh.simp_modulus(rho, 3), fixed, multigrid.Options(
        n_levels=2, dense_max=10, coarse_pcg_iters=3))
    o = simpgmg.default_options(*dims, n_levels=2, fine_prec="f64", dense_max=10, coarse_pcg_iters=3)
    h = simpgmg.setup_hierarchy(o, t64(rho), lambda_override=[lv.lam for lv in oh.levels[:-1]])
    r = workloads.random_vector(fixed.size, 6, fixed)
    z = t64(np.zeros_like(r))
    simpgmg.vcycle(h, t64(r), z)
    ref = multigrid.vcycle(oh, r)
    assert rel_err(np64(z), ref, ref) < 1e-11      # three steps: no drift beyond rounding
