"""The plain product's own launch shape (chosen beside the smoothing step's)
changes which wave computes a node, not the arithmetic."""
import numpy as np
import pytest

from tests.gpu_util import np64, t32, t64

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dims", [(17, 9, 5), (33, 14, 45)])
@pytest.mark.parametrize("prec", ["bf16", "bf16x3"])
def test_tuned_plain_product_is_bitwise_the_pinned_one(dims, prec):
    from paper_2604_26441_amd import simpgmg
    g = np.random.default_rng(4)
    opts = simpgmg.default_options(*dims, n_levels=2, fine_prec=prec)
    rho = t64(g.uniform(0.05, 1.0, np.prod(dims)))
    u = t32(g.standard_normal(3 * np.prod([d + 1 for d in dims])))

    def product(h):
        y = t32(np.zeros(u.numel()))
        simpgmg.apply_K(h, 0, prec, u, y)
        return np64(y)

    h = simpgmg.setup_hierarchy(opts, rho)
    want = product(h)                                   # the default shape
    simpgmg.autotune(h)
    assert np.array_equal(product(h), want)
    assert np.array_equal(product(simpgmg.setup_hierarchy(opts, rho)), want)   # the kept choice
    for rows, planes in ((4, 2), (8, 43)):
        simpgmg.set_launch_shape(h, prec, rows, planes)
        assert np.array_equal(product(h), want), (rows, planes)
