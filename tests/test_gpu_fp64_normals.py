"""The normals of the FP64 paths as the device computes them, against long
double from the same random words.  Bar, relative: half the logarithm's 3.2e-16,
the square root's 1.2e-16, the cosine's 3.6e-16, and the roundings of 4 dt log u
(halved), of the product, and of the quotient by sqrt(2 dt) and that root, by
which the trace is scaled back: 1.05e-15."""
import numpy as np
import pytest

from gpu_helpers import say
from paper_1504_00084_amd import workloads as W

pytestmark = pytest.mark.gpu


def normals(words):
    """Box-Muller of pairs of 32-bit words in long double."""
    m = (words >> 8 | 1).astype(np.int64)
    rad = np.sqrt(-2.0 * np.log(np.ldexp(m[:, 0].astype(np.longdouble), -24)))
    q = (m[:, 1] + (1 << 21)) >> 22
    r = np.ldexp((m[:, 1] - (q << 22)).astype(np.longdouble), -22) * (np.longdouble(2) * np.arctan(np.longdouble(1)))
    c, s = np.cos(r), np.sin(r)
    k = q & 3
    return (rad * np.choose(k, [c, -s, -c, s]), rad * np.choose(k, [s, c, -s, -c]))


def test_normals_against_long_double(oracle_lib):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1504_00084_amd import mesh_sdd as M
    M.load()
    inst = W.constant_problem(9, 2, 1, 1, 0.01, 1000, 100)   # doubly periodic: no path leaves
    inst.seed, inst.instance_id, inst.mesh_step = 2 ** 35 + 11, 9, 4
    P = oracle_lib.Problem(**inst.problem_kwargs())
    ctx = M.mesh_sdd_ctx_create(0)
    h = M.mesh_sdd_create(ctx, M.desc_for(inst, M.FP64))
    try:
        M.mesh_sdd_set_monitor(h, inst.rho)
        st = M.make_step(inst.x, inst.y, inst.bnd_t0, inst.bnd_t1, paths_per_node=100, mesh_step=inst.mesh_step)
        node = 2
        d = M.mesh_sdd_debug_paths(h, st, node, 0, 100, inst.K, trace=True)
        got = d["trace"][..., 2:].reshape(-1, 2)
        words = np.array([[oracle_lib.stream_word(P, node, p, 3 * k + w) for w in (0, 1)]
                          for p in range(100) for k in range(inst.K)], dtype=np.uint64)
        want = normals(words)
        for c in (0, 1):
            err = float(np.max(np.abs(got[:, c].astype(np.longdouble) / want[c] - 1)))
            say("normal %d: %.3e relative" % (c, err))
            assert err <= 1.05e-15
    finally:
        M.mesh_sdd_destroy(h)
        M.mesh_sdd_ctx_destroy(ctx)
