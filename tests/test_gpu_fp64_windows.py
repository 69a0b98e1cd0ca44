"""FP64 solves of grids that do not fit the LDS, on both sides of the work at
which windows of the monitor pay: launches with more run in windows, shorter
ones read global memory.  The values are the same, so the sampled nodes of a
subsampled solve (short) equal those of the full one (in windows) bit for bit;
the full one is checked against the oracle."""
import numpy as np
import pytest

from gpu_helpers import say
from test_gpu_fp64_kernel import M, ctx, problem  # noqa: F401

pytestmark = pytest.mark.gpu

# n_xi, n_eta, sub_xi, sub_eta, per_xi, per_eta, K, tau, N, stride of the short solve
CASES = [
    (143, 143, 2, 2, 0, 0, 33, 2e-3, 1984, 71),    # just past the largest table in LDS
    (145, 151, 4, 5, 1, 0, 41, 4e-3, 1000, 6),
    (289, 25, 6, 2, 0, 1, 31, 2e-2, 1700, 12),     # a long grid, wide excursions
    (25, 301, 2, 5, 1, 1, 50, 2e-2, 960, 12),
    (193, 193, 2, 3, 0, 0, 40, 4e-2, 1000, 32),    # paths that leave their windows
]


@pytest.mark.parametrize("case", CASES, ids=lambda c: "%dx%d_per%d%d_K%d_N%d" % (c[0], c[1], c[4], c[5], c[6], c[8]))
def test_windows_and_global_memory_agree(M, ctx, oracle_lib, case):  # noqa: F811
    inst = problem(*case[:9])
    N, stride = inst.n_paths, case[9]
    say("fp64 windows", case)
    P = oracle_lib.Problem(**inst.problem_kwargs())
    ora = oracle_lib.solve(P, inst.rho, inst.x, inst.y, inst.bnd_t0, inst.bnd_t1, N, threads=8)
    h = M.mesh_sdd_create(ctx, M.desc_for(inst, M.FP64))
    try:
        M.mesh_sdd_set_monitor(h, inst.rho)
        m = M.mesh_sdd_num_interface_nodes(h)
        i, j = M.mesh_sdd_interface_nodes(h)
        Px, Py = (inst.n_xi - 1) // inst.sub_xi, (inst.n_eta - 1) // inst.sub_eta
        runs = ((i % Px == 0) & (j % stride == 0)) | ((j % Py == 0) & (i % stride == 0))
        work = [n * -(-N // 64) * inst.K / 256 for n in (m, int(runs.sum()))]
        assert work[0] > 1024 >= work[1], work   # on 256 compute units, items of 64 paths
        out = []
        for s in (0, stride):
            arrs, res = M.host_result(m)
            st = M.make_step(inst.x, inst.y, inst.bnd_t0, inst.bnd_t1, paths_per_node=N, mesh_step=inst.mesh_step,
                             interface_stride=s)
            M.mesh_sdd_solve_interfaces(h, st, res)
            out.append(M.result_dict(arrs, res, m))
        full, short = out
        assert full["executed_path_steps"] == int(np.sum(ora["steps"]))
        for k in ("mean_x", "mean_y", "se_x", "se_y", "exit_frac"):
            assert np.nanmax(np.abs(full[k] - ora[k]), initial=0.0) <= 1e-9, k
            assert np.array_equal(full[k][runs], short[k][runs]), k
    finally:
        M.mesh_sdd_destroy(h)
