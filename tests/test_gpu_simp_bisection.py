"""Volume bisection of the OC update at element counts around the 1024-element
tiles of its volume pass, with and without projection, and at stop rules that
end it inside a pass of six halvings.  Reference: the oracle's bisection on
the device's own sensitivities."""
import numpy as np
import pytest

from oracle import simp
from tests.gpu_util import np64, t64

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dims", [(4, 3, 2), (16, 8, 8), (17, 9, 7), (23, 11, 9)])
@pytest.mark.parametrize("rmin,beta", [(1.5, 0.0), (1.0, 0.0), (2.3, 3.0)])
@pytest.mark.parametrize("tol,most", [(1e-9, 200), (1e-2, 200), (1e-9, 10)])
def test_bisection_matches_oracle(dims, rmin, beta, tol, most):
    from paper_2604_26441_amd import simpgmg
    n = int(np.prod(dims))
    g = np.random.default_rng(n)
    rho = g.uniform(0.05, 1.0, n)
    h = simpgmg.setup_hierarchy(simpgmg.default_options(*dims, n_levels=2, fine_prec="f64"), t64(rho))
    s = simpgmg.Simp(simpgmg.simp_params(*dims, rmin=rmin, beta=beta, volfrac=0.45, oc_tol=tol,
                                         oc_max_halvings=most))
    s.physical(t64(rho))
    dc, dv = t64(np.zeros(n)), t64(np.zeros(n))
    s.sensitivity(h, t64(g.standard_normal(h.n_dof)), dc, dv)
    x = t64(rho)
    r = s.oc_update(x)
    ref, lam = simp.oc_update(dims, rho, np64(dc), np64(dv), 0.45, 0.2, rmin, beta, 0.5, tol, most)
    # the two sum the volume in different orders (1e-15 of it), which moves the
    # multiplier by at most the last halving's width
    assert abs(r["lambda"] - lam) <= max(2.1e-9, 1e-12) * lam
    np.testing.assert_allclose(np64(x), ref, rtol=2e-9, atol=1e-14)
    assert abs(r["volume"] - simp.physical(dims, ref, rmin, beta, 0.5)[0].sum()) <= 1e-8 * n
    assert abs(r["max_change"] - np.abs(ref - rho).max()) <= 2e-9
