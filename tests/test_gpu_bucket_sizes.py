"""GPU tests of the grain bucketing at the sizes where it changes form: batches
of up to 4,096 pairs in one workgroup and more in three kernels, grain numbers
around and past a thread's registers (8,192), item tables written inside the
one-workgroup form and outside it.  The staged search is checked against the
oracle, plans against the staged search (same pools, so equal results)."""
import numpy as np
import pytest

from oracle import search as osr
from tests import parity
from tests.gpu_common import announce, exact_dist_fn, require_gpu, to_dev
from workloads import patch_mixture as pm

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nq,P,G", [(1, 1, 8), (3, 2, 1030), (1024, 4, 64), (1025, 4, 64), (256, 16, 8192),
                                    (257, 16, 8192), (60, 3, 8200), (1400, 3, 8200)])
def test_batches_around_the_bucket_forms(nq, P, G):
    torch = require_gpu()
    from paper_2606_08813_amd import hntl
    announce(f"{nq} queries x {P} probes over {G} grains: staged and plans")
    d, r, C, k = 16, 16, 12, 5
    # grains of 0 to 3 rows, and one of 700 (several block ranges)
    sizes = pm.ints(G, 51, 0, 4)
    sizes[G // 2] = 700
    off = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int64)
    N = int(off[-1])
    cent = pm.uniform_rows(G, d, 52)
    X = pm.uniform_rows(N, d, 53, lo=-0.3, hi=0.3) + np.repeat(cent, sizes, axis=0)
    basis = np.broadcast_to(np.eye(r, d, dtype=np.float32), (G, r, d)).copy()
    st = dict(centroids=cent, basis=basis, offsets=off, perm=np.arange(N, dtype=np.int32),
              codes=(X - np.repeat(cent, sizes, axis=0)).astype(np.float32), eps=np.zeros(N, np.float32))
    ix = hntl.hntl_index_create(st, X)
    Q = pm.uniform_rows(nq, d, 54)
    Qd = to_dev(Q)
    ids, dist = hntl.hntl_search(ix, Qd, P, C, k, flags=hntl.HNTL_FLAG_SYNC)
    orc = osr.search(Q, st, X, P, C, k)
    parity.check_lists(ids.cpu().numpy(), dist.cpu().numpy(), orc["ids"], orc["dist"], exact_dist_fn(X, Q))
    for sched in (None, dict(qt=1, nw=1, range=2), dict(qt=4, nw=2, range=0, proj=1),
                  dict(qt=2, nw=2, range=3, passes=2, proj=1)):
        plan = hntl.hntl_plan_create(ix, P, C, k, nq, sched=sched, flags=hntl.HNTL_FLAG_SYNC)
        for n in (nq, max(1, nq // 3)):
            a = hntl.hntl_plan_search(plan, Qd[:n].contiguous())
            assert torch.equal(a[0], ids[:n]) and torch.equal(a[1], dist[:n]), (sched, n)
        assert hntl.hntl_plan_info_get(plan)["wait_errors"] == 0
