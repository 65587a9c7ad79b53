"""The split node kernel of the matrix-free product (64 nodes per block, a wave
per element corner): partial and whole blocks, and both sides of the mesh sizes
where the gathering kernel takes over (FP32 400000 nodes, FP64 100000), against
an FP64 scatter of element products."""
import numpy as np
import pytest

import workloads
from oracle import hex8, mesh
from tests.gpu_util import np64, t32, t64

pytestmark = pytest.mark.gpu


def _reference(dims, E, u, fixed):
    """K u and |K| |u| by element products (M K M with M the free DOFs)."""
    import torch
    nx, ny, nz = dims
    i = np.arange(nx * ny * nz)
    ex, ey, ez = i % nx, (i // nx) % ny, i // (nx * ny)
    node = np.stack([(ex + (a & 1)) + (nx + 1) * ((ey + ((a >> 1) & 1)) + (ny + 1) * (ez + (a >> 2)))
                     for a in range(8)], 1)
    dof = torch.tensor((3 * node[:, :, None] + np.arange(3)).reshape(len(i), 24), device="cuda:0")
    ke = t64(hex8.ke(0.3))
    free = t64((~fixed).astype(float))
    out = []
    for k, v in ((ke, t64(u) * free), (ke.abs(), (t64(u) * free).abs())):
        y = torch.zeros(u.size, dtype=torch.float64, device="cuda:0")
        y.index_add_(0, dof.reshape(-1), ((v[dof] @ k.T) * t64(E)[:, None]).reshape(-1))
        out.append(np64(y * free))
    return out


SIZES = [("f32", (2, 2, 2)), ("f32", (7, 7, 3)), ("f32", (16, 8, 8)), ("f32", (72, 73, 72)),
         ("f32", (74, 74, 72)), ("f64", (2, 2, 2)), ("f64", (7, 7, 3)), ("f64", (45, 46, 45)),
         ("f64", (46, 46, 46))]


@pytest.mark.parametrize("prec,dims", SIZES)
def test_node_products_match_element_products(prec, dims):
    from paper_2604_26441_amd import simpgmg
    g = np.random.default_rng(2)
    rho = g.uniform(0.05, 1.0, np.prod(dims))
    fixed = workloads.cantilever_fixed(dims).astype(bool)
    u = workloads.random_vector(fixed.size, 7, fixed)
    if prec == "f32":
        u = u.astype(np.float32).astype(np.float64)
    h = simpgmg.setup_hierarchy(simpgmg.default_options(*dims, n_levels=2, fine_prec="f32"), t64(rho))
    if prec == "f64":
        simpgmg.set_launch_shape(h, "f64", 0, 0)          # the node kernel
    y = t32(np.zeros_like(u)) if prec == "f32" else t64(np.zeros_like(u))
    simpgmg.apply_K(h, 0, prec, t32(u) if prec == "f32" else t64(u), y)
    want, scale = _reference(dims, mesh.simp_modulus(rho, 3), u, fixed)
    # 24-term element products and 8 elements per node, at most 33 rounded
    # terms (FP32 6e-8, moduli and K_e rounded to FP32; FP64 1.1e-16, twice:
    # the reference rounds as well)
    tol = 2e-6 if prec == "f32" else 1e-14
    assert np.max(np.abs(np64(y) - want) / np.maximum(scale, 1e-3 * scale.max())) <= tol
