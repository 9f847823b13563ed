"""GPU test of searches of a few pairs, which scan all of them at once, against
the same queries in a larger batch, on both sides of the rule's limits (16 pairs,
2,048 rows a grain), with invalid probes and an empty grain."""
import numpy as np
import pytest

from tests.gpu_common import announce, require_gpu, to_dev
from workloads import patch_mixture as pm

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("largest", [2048, 2049])
@pytest.mark.parametrize("codes", ["fp32", "bf16", "fp8", "int16"])
def test_few_pairs_equal_a_batch(largest, codes):
    torch = require_gpu()
    from paper_2606_08813_amd import hntl
    announce(f"few pairs, grains of up to {largest} rows, {codes}")
    G, d, r, P, C, K = 12, 40, 16, 8, 70, 10
    sizes = np.array([largest, 1, 64, 65, 300, 0, 700, 128, 500, 127, 1000, 40])
    N = int(sizes.sum())
    X = pm.uniform_rows(N, d, 131)
    st = dict(centroids=pm.uniform_rows(G, d, 132), basis=pm.uniform_floats((G, r, d), 133, lo=-0.2, hi=0.2),
              offsets=np.concatenate([[0], np.cumsum(sizes)]).astype(np.int64), perm=np.arange(N, dtype=np.int32),
              codes=pm.uniform_floats((N, r), 134), eps=np.ones(N, np.float32))
    ix = hntl.hntl_index_create(st, X, codes=(codes,) if codes == "fp32" else ("fp32", codes))
    Q = to_dev(pm.uniform_rows(40, d, 135))
    probes = torch.from_numpy(np.stack([np.random.default_rng(i).permutation(G)[:P] for i in range(40)])
                              .astype(np.int32)).cuda()
    probes[::2, 0] = -1  # no nearest grain
    probes[1::3, 3] = G + 5
    for given in (None, probes):
        kw = dict(codes=codes, flags=hntl.HNTL_FLAG_SYNC)
        full = hntl.hntl_search_stages(ix, Q, P, C, K, probes_in=given, **kw)
        for nq in (1, 2, 3):
            for q0 in (0, 1, 20):
                o = hntl.hntl_search_stages(ix, Q[q0:q0 + nq].contiguous(), P, C, K,
                                            probes_in=None if given is None else given[q0:q0 + nq].contiguous(), **kw)
                for key in ("pool_ids", "pool_D", "ids", "dist"):
                    assert torch.equal(o[key], full[key][q0:q0 + nq]), (key, nq, q0)
