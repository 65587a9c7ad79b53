"""The FP64 fine product where its tiles of 8 x 8 elements make fewer rounds of 256
blocks than those of 16 x 4 (one plane per wave) and where they do not (more): the
product against the node kernel, and a V-cycle, whose smoothing steps and residuals
run the same tiles, bitwise the same with either."""
import numpy as np
import pytest

import workloads
from tests.gpu_util import np64, rel_err, t64

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dims", [(60, 60, 10), (61, 45, 12), (27, 61, 22)])
def test_both_tiles_give_the_same_bits(dims):
    from paper_2604_26441_amd import simpgmg
    rho = np.random.default_rng(1).uniform(0.05, 1.0, np.prod(dims))
    h = simpgmg.setup_hierarchy(simpgmg.default_options(*dims, n_levels=3, fine_prec="f64"), t64(rho))
    u = workloads.random_vector(h.n_dof, 9, workloads.cantilever_fixed(dims))

    def outputs(rows, planes):
        simpgmg.set_launch_shape(h, "f64", rows, planes)
        y, z = t64(np.zeros(h.n_dof)), t64(np.zeros(h.n_dof))
        simpgmg.apply_K(h, 0, "f64", t64(u), y)
        simpgmg.vcycle(h, t64(u), z)
        return np64(y), np64(z)

    want = outputs(0, 0)[0]
    got = [outputs(1, z) for z in (1, 2, 3)]
    for y, z in got[1:]:
        assert np.array_equal(y, got[0][0]) and np.array_equal(z, got[0][1])
    # 24-term products and 8 elements per node: each side rounds at most 200 terms
    # of 1.1e-16, entries of similar size
    assert rel_err(got[0][0], want, np.abs(want).max()) <= 1e-13
