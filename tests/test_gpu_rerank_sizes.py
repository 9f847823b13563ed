"""GPU test of the exact rerank at the row counts where it changes the number of
waves a row gets and the pool sizes where its rounds end, against float64."""
import numpy as np
import pytest

from tests import parity
from tests.gpu_common import announce, exact_dist_fn, require_gpu, to_dev
from tests.test_gpu_tiles import plain_index
from workloads import patch_mixture as pm

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nq", [1, 512, 513])
@pytest.mark.parametrize("d,C", [(60, 64), (128, 100), (200, 1), (768, 65), (768, 128), (33, 129), (768, 256)])
def test_rerank(nq, d, C):
    torch = require_gpu()
    from paper_2606_08813_amd import hntl
    announce(f"rerank of {nq} pools of {C}, d = {d}")
    N, k = 3000, min(10, C)
    X = pm.uniform_rows(N, d, 121)
    Q = pm.uniform_rows(nq, d, 122)
    rng = np.random.default_rng(123)
    pool = np.stack([rng.permutation(N)[:C] for _ in range(nq)]).astype(np.int32)
    pool[::3, C // 2:] = -1  # padding
    ix = plain_index(hntl, X, X[:1].copy(), r=8)
    o = hntl.hntl_search_stages(ix, to_dev(Q), 1, C, k, pool_in=to_dev(pool))
    dd = ((Q.astype(np.float64)[:, None, :] - X.astype(np.float64)[np.maximum(pool, 0)]) ** 2).sum(2)
    dd[pool < 0] = np.inf
    at = np.argsort(dd, axis=1, kind="stable")[:, :k]
    ref_d = np.take_along_axis(dd, at, 1)
    ref = np.where(np.isfinite(ref_d), np.take_along_axis(pool, at, 1), -1)
    parity.check_lists(o["ids"].cpu().numpy(), o["dist"].cpu().numpy(), ref, ref_d, exact_dist_fn(X, Q), what="rerank")
