"""Galerkin products at the edges of their kernels: meshes whose axes are even
or odd in turn (a third child in the last coarse element, at the first and at
the deeper products), with single DOFs fixed inside the body and on its last
faces besides the clamped one (coarse nodes next to a fixed DOF have a kernel of
their own), one to several 256-node blocks of coarse nodes."""
import numpy as np
import pytest

import workloads
from oracle import galerkin, mesh, multigrid
from tests.gpu_util import t64

pytestmark = pytest.mark.gpu

# all even, at all levels; one odd axis each; odd at the second level; all odd
MESHES = [(16, 8, 8), (9, 8, 8), (8, 9, 8), (8, 8, 9), (14, 10, 12), (11, 13, 9), (21, 15, 17)]


@pytest.mark.parametrize("dims", MESHES)
@pytest.mark.parametrize("pins", [0, 12, 200])
def test_stencils_match_the_oracle(dims, pins):
    import torch
    from paper_2604_26441_amd import simpgmg
    g = np.random.default_rng(pins)
    rho = g.uniform(0.05, 1.0, np.prod(dims))
    fixed = workloads.cantilever_fixed(dims).astype(bool)
    fixed[g.choice(fixed.size, pins, replace=False)] = True
    if pins:
        fixed[-3:] = [False, True, False]   # the last corner, in one direction
    oh = multigrid.build(dims, mesh.simp_modulus(rho, 3), fixed,
                         multigrid.Options(n_levels=3, lambdas=[1.0] * 2))
    h = simpgmg.setup_hierarchy(simpgmg.default_options(*dims, n_levels=3, fine_prec="f64"), t64(rho),
                                torch.tensor(fixed.astype(np.uint8), device="cuda:0"))
    for l in (1, 2):
        ref = np.transpose(galerkin.stencil_blocks(oh.levels[l].K, oh.levels[l].dims), (1, 2, 3, 0))
        # an entry is a sum of at most 8 x 8 products K_e and weights (level 1) or
        # 27 x 27 entries (level 2): each term loses a few FP64 units (1.1e-16)
        assert np.abs(h.stencil(l) - ref).max() <= 1e-13 * np.abs(ref).max(), l
