"""A mesh step whose new mesh takes the place of the old one on the device, on
the whole-grid solver: its last launch writes what other tiles may still
read.  The Dirichlet nodes hold their values at t^{n+1} from the start of such a
solve, so the result is that of a solve between separate arrays which starts
from the mesh with those values in it, bit for bit."""
import numpy as np
import pytest

from gpu_helpers import say
from paper_1504_00084_amd import workloads as W
from test_gpu_fe_tiles import inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("L", [1, 3, 8, 9, 40])
@pytest.mark.parametrize("grid", [(65, 65, 2, 2), (161, 97, 1, 1), (73, 145, 4, 1)], ids=lambda g: "%dx%d_%dx%d" % g)
def test_step_in_place(grid, L):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1504_00084_amd import mesh_sdd as M
    M.load()
    nx, ny, sx, sy = grid
    tau = L * 0.2 / ((nx - 1) ** 2 + (ny - 1) ** 2)
    rho, x, y, b = inputs(nx, ny, 0, 0, 1.0, 1.0)
    b1 = W.boundary_from_mesh(*W.uniform_mesh(nx, ny))
    say("step in place", grid, L)
    ctx = M.mesh_sdd_ctx_create(0)
    h = M.mesh_sdd_create(ctx, M.make_desc(nx, ny, sx, sy, 0, 0, K=2, tau=tau, precision=M.FP64))
    try:
        M.mesh_sdd_set_monitor(h, rho)
        m = M.mesh_sdd_num_interface_nodes(h)
        i, j = M.mesh_sdd_interface_nodes(h)

        def dev(a):
            return torch.from_numpy(np.ascontiguousarray(a)).cuda()

        opts = M.make_mp_opts(fe_substeps=L, edge_generator=0, solver=2)
        px, py, db, db1, nb = dev(x), dev(y), dev(b), dev(b1), dev(b)
        out = [torch.zeros(max(m, 1), dtype=torch.float64, device="cuda") for _ in range(5)]
        torch.cuda.synchronize()
        st = M.make_step(px, py, db, db1, paths_per_node=100)
        M.mesh_sdd_mp_step(h, st, px, py, nb, M.make_result(*out), opts)
        torch.cuda.synchronize()
        x0, y0 = x.copy(), y.copy()
        x0[j, i], y0[j, i] = out[0][:m].cpu().numpy(), out[1][:m].cpu().numpy()
        n4 = [b1[0:ny], b1[ny:2 * ny], b1[2 * ny:3 * ny], b1[3 * ny:4 * ny]]   # xi = 0: x, y; xi = 1: x, y
        x0[:, 0], y0[:, 0], x0[:, -1], y0[:, -1] = n4
        n4 = [b1[4 * ny + k * nx:4 * ny + (k + 1) * nx] for k in range(4)]     # eta = 0: x, y; eta = 1: x, y
        x0[0], y0[0], x0[-1], y0[-1] = n4
        gx, gy = torch.empty_like(px), torch.empty_like(py)
        args = [dev(x0), dev(y0), db1, out[0], out[1], gx, gy]
        torch.cuda.synchronize()
        M.mesh_sdd_subdomain_solve(h, *args, opts)
        torch.cuda.synchronize()
        assert torch.equal(px, gx) and torch.equal(py, gy)
    finally:
        M.mesh_sdd_destroy(h)
        M.mesh_sdd_ctx_destroy(ctx)
