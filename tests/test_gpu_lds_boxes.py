"""The forced LDS solve of subdomains at the edges of its workgroup: boxes whose
boundary nodes alone nearly fill it (some threads then own a boundary node
beside interior ones), boxes of the most interior nodes, and boxes around the
node counts at which a thread takes one node more."""
import numpy as np
import pytest

from gpu_helpers import say
from oracle import mp_oracle as mp
from test_gpu_fe_tiles import M, ctx, inputs  # noqa: F401

pytestmark = pytest.mark.gpu

# nx, ny, sub_xi, sub_eta, per_xi, per_eta, substeps
BOXES = [(13, 501, 4, 1, 0, 0, 5), (501, 13, 1, 4, 0, 1, 5), (31, 481, 10, 1, 1, 0, 6), (481, 31, 1, 10, 0, 0, 4),
         (7, 509, 3, 1, 0, 0, 3), (509, 5, 1, 2, 0, 0, 3), (257, 33, 2, 2, 0, 0, 9), (33, 257, 2, 2, 0, 1, 9),
         (129, 129, 2, 2, 0, 0, 7), (131, 129, 2, 2, 0, 0, 7), (81, 81, 2, 2, 1, 1, 5), (65, 69, 2, 2, 0, 0, 5),
         (97, 97, 3, 3, 0, 0, 5), (33, 449, 2, 2, 0, 0, 4), (73, 109, 1, 3, 0, 0, 5), (109, 109, 2, 2, 1, 0, 6)]


@pytest.mark.parametrize("case", BOXES, ids=lambda c: "%dx%d_%dx%d_per%d%d_L%d" % c)
def test_forced_lds_solve_equals_oracle(M, ctx, case):  # noqa: F811
    nx, ny, sx, sy, px, py, L = case
    Lx, Ly, tau = 1.0, 2.0, L * 0.2 / ((nx - 1) ** 2 + (ny - 1) ** 2)
    rho, x, y, b = inputs(nx, ny, px, py, Lx, Ly)
    say("LDS boxes", case)
    h = M.mesh_sdd_create(ctx, M.make_desc(nx, ny, sx, sy, px, py, K=1, Lx=Lx, Ly=Ly, tau=tau, precision=M.FP64))
    try:
        M.mesh_sdd_set_monitor(h, rho)
        m = M.mesh_sdd_num_interface_nodes(h)
        i, j = M.mesh_sdd_interface_nodes(h)
        rng = np.random.default_rng(2)
        ix = np.concatenate([x[j, i] + 1e-3 * rng.standard_normal(m), [0.0]])
        iy = np.concatenate([y[j, i] + 1e-3 * rng.standard_normal(m), [0.0]])
        wx, wy = mp.subdomain_solve(rho, x, y, b, ix[:m], iy[:m], tau, sx, sy, px, py, Lx, Ly, substeps=L)
        for solver in (1, 0):
            gx, gy = np.empty_like(x), np.empty_like(y)
            M.mesh_sdd_subdomain_solve(h, x, y, b, ix, iy, gx, gy, M.make_mp_opts(fe_substeps=L, solver=solver))
            assert np.array_equal(gx, wx) and np.array_equal(gy, wy), solver
    finally:
        M.mesh_sdd_destroy(h)
