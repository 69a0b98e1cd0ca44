"""Result arrays of a context on a stream of the caller's: work that the
default stream still has to do on them (here a fill behind a long wait) comes
before the results, on whatever stream the solve runs; a batch and a mesh step
likewise."""
import numpy as np
import pytest

from paper_1504_00084_amd import workloads as W

pytestmark = pytest.mark.gpu

FIELDS = 5


@pytest.mark.parametrize("call", ["solve", "batch", "step"])
@pytest.mark.parametrize("own", [True, False], ids=["own", "supplied"])
def test_results_follow_default_stream_work(call, own):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1504_00084_amd import mesh_sdd as M
    M.load()
    side = torch.cuda.Stream()
    inst = W.config1(500)
    inst.K = 20
    ctx = M.mesh_sdd_ctx_create(0, 0, None if own else side.cuda_stream)
    h = M.mesh_sdd_create(ctx, M.desc_for(inst, M.FP32))
    try:
        M.mesh_sdd_set_monitor(h, inst.rho)
        m = M.mesh_sdd_num_interface_nodes(h)
        dev = [torch.from_numpy(np.ascontiguousarray(a)).cuda() for a in (inst.x, inst.y, inst.bnd_t0, inst.bnd_t1)]
        torch.cuda.synchronize()
        st = M.make_step(*dev, paths_per_node=500)

        def run(busy):
            out = [torch.empty(m, dtype=torch.float64, device="cuda") for _ in range(FIELDS)]
            mesh = [torch.empty_like(a) for a in (dev[0], dev[1], dev[3])]
            torch.cuda.synchronize()
            if busy:
                torch.cuda._sleep(200_000_000)   # the default stream is behind
                for a in out:
                    a.fill_(7.0)
            res = M.make_result(*out)
            if call == "solve":
                M.mesh_sdd_solve_interfaces(h, st, res)
            elif call == "batch":
                M.mesh_sdd_solve_batch([h], [st], [res])
            else:
                M.mesh_sdd_mp_step(h, st, *mesh, res, M.make_mp_opts(edge_generator=0))
            torch.cuda.synchronize()
            return [a.cpu().numpy() for a in out]

        want = run(False)
        got = run(True)
        assert all(np.all(np.isfinite(a)) for a in want)
        for a, b in zip(want, got):
            assert np.array_equal(a, b)
    finally:
        M.mesh_sdd_destroy(h)
        M.mesh_sdd_ctx_destroy(ctx)
