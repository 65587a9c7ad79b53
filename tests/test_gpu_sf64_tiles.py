"""Sum/difference-basis products on grids around the edges of both tile shapes
(16 x 4 elements owning 15 x 3 nodes, 8 x 8 owning 7 x 7): the fine operator
against the node kernel, the level-1 products against the stored stencil."""
import numpy as np
import pytest

import workloads
from tests.gpu_util import np64, rel_err, t64

pytestmark = pytest.mark.gpu

# nodes per axis in x and y: 7 x 7, 8 x 7, 14 x 14, 15 x 3, 16 x 4, 31 x 31, 29 x 10
GRIDS = [(6, 6, 4), (7, 6, 5), (13, 13, 3), (14, 2, 6), (15, 3, 4), (30, 30, 5), (28, 9, 6)]


@pytest.mark.parametrize("dims", GRIDS)
@pytest.mark.parametrize("level", [0, 1])
def test_tiles_match_the_other_kernels(dims, level):
    from paper_2604_26441_amd import simpgmg
    mesh_dims = tuple(d << level for d in dims)
    rho = np.random.default_rng(1).uniform(0.05, 1.0, np.prod(mesh_dims))
    opts = simpgmg.default_options(*mesh_dims, n_levels=3 if level else 2, fine_prec="f64", stencil_form=3)
    h = simpgmg.setup_hierarchy(opts, t64(rho))
    n = 3 * np.prod([d + 1 for d in dims])
    u = workloads.random_vector(n, 9, workloads.cantilever_fixed(dims))
    variant = "level1" if level else "f64"

    def product(rows, planes):
        simpgmg.set_launch_shape(h, variant, rows, planes)
        y = t64(np.zeros(n))
        simpgmg.apply_K(h, level, "f64", t64(u), y)
        return np64(y)

    want = product(0, 1 if level else 0)          # the stored stencil; the node kernel
    got = [product(1, z) for z in (1, 2, 5)]
    for y in got[1:]:
        assert np.array_equal(y, got[0])          # the chunk length moves work only
    # 24-term products and 8 elements (level 1: 64 children) per node: each
    # side rounds at most 200 terms of 1.1e-16, entries of similar size
    assert rel_err(got[0], want, np.abs(want).max()) <= 1e-13
