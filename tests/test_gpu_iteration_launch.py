"""The PCG iteration on both sides of the size from which it is launched kernel
by kernel instead of replayed from a graph (100,000 DOFs).  The kernels and
their arguments are the same, so every output has to be bitwise that of the
solver that never uses a graph: on a first solve, after new moduli, with the
Jacobi preconditioner, and where a large mesh keeps its graph (the iterative
coarsest solve, the W-cycle)."""
import numpy as np
import pytest

import workloads

pytestmark = pytest.mark.gpu

CASES = [((32, 31, 30), {}), ((32, 32, 31), {}), ((32, 32, 31), {"dense_max": 100, "coarse_pcg_iters": 20}),
         ((32, 32, 31), {"cycle_gamma": 2}), ((40, 33, 36), {"fine_prec": "f64"})]


@pytest.mark.parametrize("dims,opts", CASES)
def test_iteration_equals_direct_launches(dims, opts):
    import torch
    from paper_2604_26441_amd import simpgmg

    def t64(a):
        return torch.tensor(a, dtype=torch.float64, device="cuda:0")

    rho = np.random.default_rng(8).uniform(0.2, 1.0, np.prod(dims))
    f = workloads.edge_load(dims)
    out = []
    for g in (0, 1):
        o = simpgmg.default_options(*dims, **{"n_levels": 3, "fine_prec": "bf16x3", "use_graphs": g, **opts})
        h = simpgmg.setup_hierarchy(o, t64(rho))
        got = []
        for scale, precond, rtol in ((1.0, 2, 1e-8), (1.0, 1, 1e-2), (0.6, 2, 1e-8), (0.59, 2, 1e-8)):
            if scale != 1.0:
                simpgmg.update_moduli(h, t64(scale * rho))
            u = t64(np.zeros_like(f))
            r = simpgmg.pcg_solve(h, t64(f), u, rtol=rtol, maxit=60, precond=precond, history_cap=64)
            got.append((r["status"], r["iters"], r["history"], u.cpu().numpy()))
        h.close()
        out.append(got)
    for a, b in zip(*out):
        assert a[:3] == b[:3]
        assert np.array_equal(a[3], b[3])
