"""The forward-Euler solves at the edges of their kernels: grids around the
tile size and its rim, periodic grids shorter than a tile with its rim, grids
whose cell counts are powers of two (no divisions) and not, subdomains of
one cell, subdomains around the row counts per thread and the sizes that one
workgroup holds, and substep counts around those of one launch."""
import numpy as np
import pytest

from gpu_helpers import say
from oracle import mp_oracle as mp
from paper_1504_00084_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def M():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1504_00084_amd import mesh_sdd
    mesh_sdd.load()
    return mesh_sdd


@pytest.fixture(scope="module")
def ctx(M):
    c = M.mesh_sdd_ctx_create(0)
    yield c
    M.mesh_sdd_ctx_destroy(c)


def inputs(nx, ny, px, py, Lx, Ly):
    rng = np.random.default_rng([nx, ny, px, py])
    xi, eta = np.meshgrid(np.arange(nx) / (nx - 1), np.arange(ny) / (ny - 1))
    rho = 1.3 + np.sin(2 * np.pi * xi + 0.3) * np.cos(2 * np.pi * eta)
    x = Lx * xi + 0.02 * np.sin(2 * np.pi * xi) * np.cos(2 * np.pi * eta) * rng.uniform(0.5, 1.0)
    y = Ly * eta + 0.02 * np.sin(2 * np.pi * eta) * np.cos(2 * np.pi * xi) * rng.uniform(0.5, 1.0)
    return rho, np.ascontiguousarray(x), np.ascontiguousarray(y), W.boundary_from_mesh(x, y)


# nx, ny, per_xi, per_eta, substeps
SINGLE = [(4, 4, 0, 0, 1), (18, 18, 0, 0, 8), (19, 35, 0, 0, 9), (33, 34, 0, 0, 16), (17, 17, 1, 1, 17),
          (5, 40, 1, 0, 10), (16, 5, 0, 1, 1), (18, 33, 1, 1, 2), (33, 65, 1, 0, 25), (65, 17, 0, 1, 7)]


@pytest.mark.parametrize("case", SINGLE, ids=lambda c: "%dx%d_per%d%d_L%d" % c)
def test_single_domain_equals_oracle(M, ctx, case):
    """Every update is the oracle's sequence of IEEE operations (the divisions
    by powers of two are exact scalings), so the meshes are equal."""
    nx, ny, px, py, L = case
    Lx, Ly, tau = 1.5, 0.75, L * 0.2 / ((nx - 1) ** 2 + (ny - 1) ** 2)
    rho, x, y, b = inputs(nx, ny, px, py, Lx, Ly)
    say("single domain", case)
    h = M.mesh_sdd_create(ctx, M.make_desc(nx, ny, 1, 1, px, py, K=1, Lx=Lx, Ly=Ly, tau=tau, precision=M.FP64))
    try:
        M.mesh_sdd_set_monitor(h, rho)
        gx, gy = np.empty_like(x), np.empty_like(y)
        M.mesh_sdd_single_domain_solve(h, x, y, b, gx, gy, M.make_mp_opts(fe_substeps=L))
        wx, wy = mp.single_domain_solve(rho, x, y, b, tau, px, py, Lx, Ly, substeps=L)
        assert np.array_equal(gx, wx) and np.array_equal(gy, wy)
    finally:
        M.mesh_sdd_destroy(h)


# nx, ny, sub_xi, sub_eta, per_xi, per_eta, substeps
BOXES = [(9, 9, 8, 2, 0, 0, 5), (9, 25, 2, 8, 0, 0, 9), (33, 33, 4, 4, 1, 1, 11), (37, 25, 4, 3, 0, 1, 8),
         (129, 65, 2, 1, 0, 0, 10), (73, 145, 1, 2, 0, 0, 9), (67, 23, 2, 2, 1, 0, 17), (97, 97, 1, 1, 0, 0, 3),
         (69, 31, 2, 2, 1, 1, 9), (21, 73, 2, 2, 1, 1, 9)]   # two rows of a column per thread


@pytest.mark.parametrize("solver", [0, 2], ids=["auto", "sweep"])
@pytest.mark.parametrize("case", BOXES, ids=lambda c: "%dx%d_%dx%d_per%d%d_L%d" % c)
def test_subdomains_equal_oracle(M, ctx, case, solver):
    nx, ny, sx, sy, px, py, L = case
    Lx, Ly, tau = 1.0, 2.0, L * 0.2 / ((nx - 1) ** 2 + (ny - 1) ** 2)
    rho, x, y, b = inputs(nx, ny, px, py, Lx, Ly)
    say("subdomains", case, solver)
    h = M.mesh_sdd_create(ctx, M.make_desc(nx, ny, sx, sy, px, py, K=1, Lx=Lx, Ly=Ly, tau=tau, precision=M.FP64))
    try:
        M.mesh_sdd_set_monitor(h, rho)
        m = M.mesh_sdd_num_interface_nodes(h)
        i, j = M.mesh_sdd_interface_nodes(h)
        rng = np.random.default_rng(1)
        ix = np.concatenate([x[j, i] + 1e-3 * rng.standard_normal(m), [0.0]])
        iy = np.concatenate([y[j, i] + 1e-3 * rng.standard_normal(m), [0.0]])
        gx, gy = np.empty_like(x), np.empty_like(y)
        M.mesh_sdd_subdomain_solve(h, x, y, b, ix, iy, gx, gy, M.make_mp_opts(fe_substeps=L, solver=solver))
        wx, wy = mp.subdomain_solve(rho, x, y, b, ix[:m], iy[:m], tau, sx, sy, px, py, Lx, Ly, substeps=L)
        assert np.array_equal(gx, wx) and np.array_equal(gy, wy)
    finally:
        M.mesh_sdd_destroy(h)


@pytest.mark.parametrize("case", [(4, 65, 0, 0), (64, 65, 0, 0), (65, 66, 0, 0), (129, 257, 0, 0), (1025, 5, 0, 0),
                                  (5, 1026, 0, 0), (257, 64, 1, 0), (66, 1030, 0, 1)],
                         ids=lambda c: "%dx%d_per%d%d" % c)
def test_edge_generator_equals_oracle(M, ctx, case):
    nx, ny, px, py = case
    Lx, Ly, tau = 1.0, 2.0, 4.0 / max(nx, ny) ** 2
    rho, x, y, b = inputs(nx, ny, px, py, Lx, Ly)
    say("edges", case)
    h = M.mesh_sdd_create(ctx, M.make_desc(nx, ny, 1, 1, px, py, K=1, Lx=Lx, Ly=Ly, tau=tau, precision=M.FP64))
    try:
        M.mesh_sdd_set_monitor(h, rho)
        got = np.empty_like(b)
        M.mesh_sdd_edge_generate(h, b, got)
        assert np.array_equal(got, mp.edge_generate(rho, b, tau, px, py, Lx, Ly))
    finally:
        M.mesh_sdd_destroy(h)
