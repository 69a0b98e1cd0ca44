"""Small requests run in slices of 64 paths, whose values the finalize sums as
whole chunks: the same bits as a context whose memory budget leaves no room for
the slices' records, which runs whole chunks; also where every path of a node
ends at the same value, whose spread is rounding alone."""
import numpy as np
import pytest

from gpu_helpers import say
from test_gpu_fp64_kernel import problem

pytestmark = pytest.mark.gpu

FIELDS = ("mean_x", "mean_y", "se_x", "se_y", "exit_frac")

# n_xi, n_eta, sub_xi, sub_eta, per_xi, per_eta, K, tau, paths, paths per chunk (0: the default)
CASES = [
    (17, 17, 2, 2, 0, 0, 80, 0.02, 20000, 0),
    (17, 17, 4, 4, 1, 0, 64, 50.0, 16384, 192),  # long substeps; 86 chunks of three slices
    (33, 17, 2, 4, 1, 0, 65, 50.0, 8257, 256),   # a last chunk of two slices, the second of one path
    (17, 33, 4, 2, 0, 1, 100, 0.05, 8191, 128),
    (161, 49, 4, 2, 1, 1, 66, 0.01, 4100, 0),     # in windows
]


@pytest.mark.parametrize("case", CASES, ids=lambda c: "%dx%d_per%d%d_N%d_c%d" % (c[0], c[1], c[4], c[5], c[8], c[9]))
def test_slices_equal_whole_chunks(case):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1504_00084_amd import mesh_sdd as M
    M.load()
    inst = problem(*case[:9])
    out = []
    for budget in (0, 3 << 20):
        ctx = M.mesh_sdd_ctx_create(0, hbm_budget_bytes=budget)
        h = M.mesh_sdd_create(ctx, M.desc_for(inst, M.FP32))
        try:
            if case[9]:
                M.mesh_sdd_set_launch(ctx, M.make_launch(chunk_paths=case[9]))
            M.mesh_sdd_set_monitor(h, inst.rho)
            m = M.mesh_sdd_num_interface_nodes(h)
            assert m * (inst.n_paths // 64) * 528 > 3 << 20   # the records of the slices
            for n in (inst.n_paths, 129, 64, 1):
                st = M.make_step(inst.x, inst.y, inst.bnd_t0, inst.bnd_t1, paths_per_node=n, mesh_step=inst.mesh_step)
                arrs, res = M.host_result(m)
                M.mesh_sdd_solve_interfaces(h, st, res)
                out.append(M.result_dict(arrs, res, m))
        finally:
            M.mesh_sdd_destroy(h)
            M.mesh_sdd_ctx_destroy(ctx)
    for a, b in zip(out[:4], out[4:]):
        assert a["executed_path_steps"] == b["executed_path_steps"]
        for k in FIELDS:
            assert np.array_equal(a[k], b[k], equal_nan=True), k
    say("%s: slices == whole chunks, %d nodes" % (case[:2], m))
