"""The table kernel's two forms on both sides of the grid size that parts them
(all three fields with their differences along xi in LDS up to 6826 nodes, two
fields above): the same bits as the cell-record kernel, which reads no table."""
import numpy as np
import pytest

from gpu_helpers import say
from test_gpu_fp64_kernel import problem

pytestmark = pytest.mark.gpu

FIELDS = ("mean_x", "mean_y", "se_x", "se_y", "exit_frac", "executed_path_steps")

# n_xi, n_eta, sub_xi, sub_eta, per_xi, per_eta, K, tau, N
CASES = [
    (4, 4, 1, 3, 0, 0, 5, 0.01, 65),
    (83, 82, 2, 3, 0, 0, 30, 0.05, 200),         # 6806 nodes: the last square grid of three fields
    (83, 83, 2, 2, 1, 1, 30, 0.05, 130),         # 6889: two fields
    (1706, 4, 5, 1, 0, 0, 12, 0.02, 100),        # 6824: the longest rows
    (4, 1706, 1, 5, 0, 1, 12, 0.02, 100),        # and the longest columns
    (41, 33, 4, 2, 1, 0, 37, 0.05, 300),
    (33, 41, 2, 4, 1, 1, 37, 0.05, 300),
    (33, 17, 4, 2, 0, 0, 3, 0.3, 1000),          # dt = 0.1: all four sides in the bridge test
    (17, 33, 2, 4, 1, 0, 2, 0.5, 700),
    (33, 33, 2, 2, 0, 1, 2, 0.5, 129),
]


@pytest.mark.parametrize("case", CASES, ids=lambda c: "%dx%d_per%d%d_K%d_N%d" % (c[0], c[1], c[4], c[5], c[6], c[8]))
def test_table_forms_equal_the_record_kernel(case):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1504_00084_amd import mesh_sdd as M
    M.load()
    inst = problem(*case)
    ctx = M.mesh_sdd_ctx_create(0)
    h = M.mesh_sdd_create(ctx, M.desc_for(inst, M.FP32))
    try:
        M.mesh_sdd_set_monitor(h, inst.rho)
        m = M.mesh_sdd_num_interface_nodes(h)
        st = M.make_step(inst.x, inst.y, inst.bnd_t0, inst.bnd_t1, paths_per_node=inst.n_paths, mesh_step=inst.mesh_step)
        out = []
        for launch in (None, M.make_launch(monitor_table=1)):
            M.mesh_sdd_set_launch(ctx, launch)
            level = M.mesh_sdd_get_launch(h).table_level
            assert level == (0 if launch else 2)
            arrs, res = M.host_result(m)
            M.mesh_sdd_solve_interfaces(h, st, res)
            out.append(M.result_dict(arrs, res, m))
    finally:
        M.mesh_sdd_destroy(h)
        M.mesh_sdd_ctx_destroy(ctx)
    for k in FIELDS:
        assert np.array_equal(out[0][k], out[1][k]), k
    say("%s: table == records, %d path-steps" % (case[:2], out[0]["executed_path_steps"]))
