"""True residual of the staged batch (on the tiles of the iteration's K p) from a
given start, without an iteration: meshes on and off the tile edges."""
import numpy as np
import pytest

import workloads
from oracle import mesh
from tests.gpu_util import t64

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dims", [[(6, 6, 4), (14, 2, 6), (16, 12, 10)], [(9, 7, 5), (30, 6, 7), (8, 8, 8)]])
def test_residual_of_a_start_matches_the_oracle(dims):
    from paper_2604_26441_amd import simpgmg
    rng = np.random.default_rng(8)
    rhos = [rng.uniform(0.1, 1.0, np.prod(d)) for d in dims]
    opts = [simpgmg.default_options(*d, n_levels=2, fine_prec="bf16x3") for d in dims]
    b = simpgmg.setup_batch(opts, [t64(r) for r in rhos])
    fixed = [workloads.cantilever_fixed(d).astype(bool) for d in dims]
    f = [workloads.random_vector(x.size, 2, x) for x in fixed]
    u = [workloads.random_vector(x.size, 3, x) for x in fixed]
    res, _ = simpgmg.pcg_solve_batch(b, [0, 1, 2], [t64(v) for v in f], [t64(v) for v in u], rtol=1e-12,
                                     maxit=0, staged=True)
    for k, d in enumerate(dims):
        r = f[k] - mesh.assemble(d, mesh.simp_modulus(rhos[k], 3), fixed=fixed[k]) @ u[k]
        want = np.linalg.norm(r) / np.linalg.norm(f[k])
        # sums of at most 6000 squares of residuals that are good to 200 x 1.1e-16
        assert abs(res[k]["rel_res_recur"] - want) <= 1e-12 * want
        assert res[k]["status"] == "maxit" and res[k]["iters"] == 0
