"""GPU test of the schedule that a plan takes by default: tiles of four pairs where
many short items of one would wait for their turn, single pairs elsewhere, the
results those of a search either way."""
import numpy as np
import pytest

from tests.gpu_common import announce, require_gpu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("rows,G,nq,P,qt", [
    (20, 300, 1030, 8, 4), (20, 300, 1000, 8, 1),  # short grains: from 8,192 pairs
    (128, 300, 1030, 8, 4), (129, 300, 1030, 8, 1),
    (150, 600, 2048, 4, 4), (150, 600, 2047, 4, 1),  # 13.6 pairs a grain
    (150, 64, 256, 8, 4), (150, 64, 255, 8, 1),  # 32 pairs a grain
    (10, 4000, 300, 2, 1)])  # fewer pairs than grains
def test_tiles_by_pairs(rows, G, nq, P, qt):
    torch = require_gpu()
    from paper_2606_08813_amd import hntl
    announce(f"default plan of {nq} x {P} pairs over {G} grains of {rows} rows")
    d, r, N = 16, 16, rows * G
    g = torch.Generator(device="cuda").manual_seed(G)
    cent = 3.0 * torch.randn(G, d, device="cuda", generator=g)
    z = torch.randn(N, r, device="cuda", generator=g)
    X = cent.repeat_interleave(rows, 0) + z
    W = torch.eye(d, device="cuda").expand(G, r, d).contiguous()
    st = dict(centroids=cent, basis=W, offsets=rows * np.arange(G + 1, dtype=np.int64), perm=np.arange(N, dtype=np.int32),
              codes=z, eps=torch.zeros(N, device="cuda"))
    ix = hntl.hntl_index_create(st, X)
    Q = X[torch.randint(0, N, (nq,), device="cuda", generator=g)].contiguous()
    plan = hntl.hntl_plan_create(ix, P, 16, 10, nq)
    assert hntl.hntl_plan_info_get(plan)["sched"]["qt"] == qt
    got = hntl.hntl_plan_search(plan, Q)
    want = hntl.hntl_search(ix, Q, P, 16, 10, flags=hntl.HNTL_FLAG_SYNC)
    assert torch.equal(got[0], want[0]) and torch.equal(got[1], want[1])
