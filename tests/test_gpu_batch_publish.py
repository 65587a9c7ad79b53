"""The host loop of the staged batch against the same items in one graph launch,
whose decisions are taken on the device: the flags and scalars cross the bus in
one block's strides (256 threads; 2 flags and 8 scalars per item), with one
item, on both sides of a stride and over several.  The items differ, so they
stop at different iterations and every pass has other flags."""
import numpy as np
import pytest

import workloads
from tests.gpu_util import t64, np64

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 32, 33, 128, 129, 300])
def test_host_loop_equals_one_launch(n):
    from paper_2604_26441_amd import simpgmg
    dims = [(8, 4, 4), (12, 6, 6), (9, 7, 5)]
    rng = np.random.default_rng(5)
    opts = [simpgmg.default_options(*d, n_levels=2, fine_prec="bf16x3") for d in dims]
    b = simpgmg.setup_batch(opts, [t64(rng.uniform(0.05, 1.0, np.prod(d))) for d in dims])
    sys_of = [k % 3 for k in range(n)]
    fixed = [workloads.cantilever_fixed(d).astype(bool) for d in dims]
    f = []
    for k, s in enumerate(sys_of):
        v = workloads.random_vector(fixed[s].size, 10 + k, fixed[s])
        if k % 7 == 3:
            v[:] = 0.0                       # stops before the first iteration
        elif k % 5 == 2:
            v = workloads.edge_load(dims[s])
        f.append(t64(v))
    out = []
    for staged in (True, True, False):       # the second solve starts on the first one's buffers
        u = [t64(np.zeros(x.numel())) for x in f]
        if staged:
            res, _ = simpgmg.pcg_solve_batch(b, sys_of, f, u, rtol=1e-7, maxit=40, staged=True)
        else:
            res, _, _ = simpgmg.pcg_solve_batch_graph(b, sys_of, f, u, rtol=1e-7, maxit=40, steps=40)
        out.append((res, [np64(x) for x in u]))
    for res, u in out[1:]:
        for k in range(n):
            assert res[k]["status"] == out[0][0][k]["status"] == "converged"
            assert res[k]["iters"] == out[0][0][k]["iters"]
            assert np.array_equal(u[k], out[0][1][k])
