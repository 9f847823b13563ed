"""GPU tests of the start of a plan's run: queries in any alignment, every form of
routing operand, batches below the plan's size in any order, results in the
caller's buffers and in the plan's own, and nothing past the batch written."""
import numpy as np
import pytest

from oracle import router as orr
from tests.gpu_common import announce, require_gpu
from workloads import patch_mixture as pm

pytestmark = pytest.mark.gpu

N, G, R, P, C, K = 6000, 40, 16, 4, 32, 8


def view_at(torch, address, shape, dtype):
    """A CUDA tensor over a plan's buffer."""
    class Holder:
        __cuda_array_interface__ = dict(data=(address, False), shape=shape, version=3,
                                        typestr="<i4" if dtype == torch.int32 else "<f4")
    return torch.as_tensor(Holder(), device="cuda")


@pytest.mark.parametrize("d", [16, 264, 1032])  # a lane's share of a row: none to several rounds
@pytest.mark.parametrize("route,flags", [("centroid", 0), ("centroid", 32), ("centroid", 128), ("learned", 0)],
                         ids=["fp32", "bf16x3", "bf16", "learned"])
def test_runs_equal_searches(d, route, flags):
    torch = require_gpu()
    from paper_2606_08813_amd import hntl
    announce(f"plan runs, d = {d}, {route} {flags}")
    g = torch.Generator(device="cuda").manual_seed(d)
    X = torch.randn(N, d, device="cuda", generator=g)
    ix = hntl.hntl_build(X, G, R, seed=1, kmeans_iters=2)
    if route == "learned":
        p = {k: v.astype(np.float32) for k, v in orr.init_params((d, 16, 24, G), seed=4).items()}
        hntl.hntl_router_set(ix, p, pm.uniform_rows(1, d, 5)[0], np.linspace(0.5, 2.0, d).astype(np.float32))
    sync = hntl.HNTL_FLAG_SYNC
    max_nq = 70
    for graph in (True, False):
        plan = hntl.hntl_plan_create(ix, P, C, K, max_nq, flags=flags | sync, route=route, graph=graph)
        _, ia, da = hntl.hntl_plan_buffers(plan)
        own_i, own_d = view_at(torch, ia, (max_nq, K), torch.int32), view_at(torch, da, (max_nq, K), torch.float32)
        for nq, shift in ((max_nq, 0), (1, 1), (17, 2), (max_nq, 3), (16, 0), (5, 1)):
            buf = torch.randn(nq * d + 4, device="cuda", generator=g)
            Q = buf[shift:shift + nq * d].view(nq, d)
            ids = torch.full((nq + 2, K), -5, dtype=torch.int32, device="cuda")
            dist = torch.full((nq + 2, K), -5.0, device="cuda")
            hntl.hntl_plan_search(plan, Q, out=(ids, dist))
            want = hntl.hntl_search(ix, Q.clone(), P, C, K, flags=flags | sync, route=route)
            assert torch.equal(ids[:nq], want[0]) and torch.equal(dist[:nq], want[1]), (graph, nq, shift)
            assert (ids[nq:] == -5).all() and (dist[nq:] == -5.0).all()
            assert torch.equal(own_i[:nq], ids[:nq]) and torch.equal(own_d[:nq], dist[:nq])
            assert (own_i[nq:] == -1).all()
            hntl.hntl_plan_run(plan, nq)  # the same queries again, in the plan's buffers only
            assert torch.equal(own_i[:nq], ids[:nq])
