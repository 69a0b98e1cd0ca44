"""The FP64 path kernel at the edges of its forms: grids on both sides of the
141 nodes whose padded monitor table fits the LDS whole, windows that meet
the grid's border, rectangular grids, every periodicity, path counts below,
at and past a wave and an item, substep counts that are no multiple of four,
substeps long enough for the far side of an axis in the bridge test."""
import numpy as np
import pytest

from gpu_helpers import say
from paper_1504_00084_amd import workloads as W

pytestmark = pytest.mark.gpu

# n_xi, n_eta, sub_xi, sub_eta, per_xi, per_eta, K, tau, N
CASES = [
    (4, 4, 1, 3, 0, 0, 1, 0.02, 1),
    (141, 141, 2, 2, 0, 0, 5, 2e-3, 65),        # the largest square table in LDS
    (143, 141, 2, 2, 0, 0, 6, 2e-3, 63),        # just past it: windows
    (142, 149, 3, 4, 1, 0, 7, 4e-3, 130),
    (289, 25, 6, 2, 0, 1, 30, 2e-2, 257),       # a long grid in windows, wide excursions
    (25, 301, 2, 5, 1, 1, 31, 2e-2, 64),
    (193, 193, 2, 3, 0, 0, 40, 4e-2, 40),       # paths that leave their windows
    (33, 17, 4, 2, 0, 0, 3, 0.3, 1000),         # dt = 0.1: both sides of an axis in the bridge test
    (17, 33, 2, 4, 1, 0, 2, 0.5, 700),
]


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


def problem(n_xi, n_eta, sub_xi, sub_eta, per_xi, per_eta, K, tau, N):
    inst = W.constant_problem(9, 2, per_xi, per_eta, tau, K, N)
    x, y = W.uniform_mesh(n_xi, n_eta)
    x += 0.02 * np.sin(2 * np.pi * x) * np.cos(2 * np.pi * y)
    y += 0.02 * np.sin(2 * np.pi * y) * np.cos(2 * np.pi * x)
    rho = 1.5 + np.sin(2 * np.pi * x) * np.cos(2 * np.pi * y) + 0.3 * np.cos(2 * np.pi * y) ** 2
    inst.n_xi, inst.n_eta, inst.sub_xi, inst.sub_eta = n_xi, n_eta, sub_xi, sub_eta
    inst.x, inst.y, inst.rho = x, y, np.ascontiguousarray(rho)
    inst.bnd_t0 = W.boundary_from_mesh(x, y)
    inst.bnd_t1 = inst.bnd_t0.copy()
    inst.seed, inst.instance_id, inst.mesh_step = 2 ** 40 + 7, 3, 5
    return inst


@pytest.mark.parametrize("case", CASES, ids=lambda c: "%dx%d_per%d%d_K%d_N%d" % (c[0], c[1], c[4], c[5], c[6], c[8]))
def test_fp64_kernel_against_oracle_and_its_own_paths(M, ctx, oracle_lib, case):
    """Every node against the oracle to 1e-9 (the bar of the FP64 kernel), and
    some nodes against the mean of their single paths, which read the
    monitor from global memory with the same arithmetic: they differ by the
    order of the sums only, at most N roundings of the largest |v - v_ref|."""
    inst = problem(*case)
    N = inst.n_paths
    say("fp64 kernel", case)
    P = oracle_lib.Problem(**inst.problem_kwargs())
    ora = oracle_lib.solve(P, inst.rho, inst.x, inst.y, inst.bnd_t0, inst.bnd_t1, N, threads=8)
    h = M.mesh_sdd_create(ctx, M.desc_for(inst, M.FP64))
    try:
        M.mesh_sdd_set_monitor(h, inst.rho)
        m = M.mesh_sdd_num_interface_nodes(h)
        arrs, res = M.host_result(m)
        st = M.make_step(inst.x, inst.y, inst.bnd_t0, inst.bnd_t1, paths_per_node=N, mesh_step=inst.mesh_step)
        M.mesh_sdd_solve_interfaces(h, st, res)
        g = M.result_dict(arrs, res, m)
        assert g["executed_path_steps"] == int(np.sum(ora["steps"]))
        for k in ("mean_x", "mean_y", "se_x", "se_y", "exit_frac"):
            assert np.array_equal(np.isnan(g[k]), np.isnan(ora[k])), k
            assert np.nanmax(np.abs(g[k] - ora[k]), initial=0.0) <= 1e-9, k
        i, j = M.mesh_sdd_interface_nodes(h)
        for r in sorted({0, m // 3, m - 1}):
            d = M.mesh_sdd_debug_paths(h, st, r, 0, N, inst.K)
            for v, mean, ref in (("vx", "mean_x", inst.x), ("vy", "mean_y", inst.y)):
                dv = d[v] - ref[j[r], i[r]]
                bar = (N + 4) * 2.0 ** -53 * np.max(np.abs(dv)) + 2.0 ** -51
                assert abs(ref[j[r], i[r]] + dv.mean() - g[mean][r]) <= bar, (r, v)
    finally:
        M.mesh_sdd_destroy(h)
