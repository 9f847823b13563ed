"""GPU tests of the k-means++ seeding kernels at the sizes where their blocks end
(16 rows per tile, 256 per block, 64 block sums at a time, odd depths, the direct
distances of very few rows): clusters far apart each get one centroid."""
import numpy as np
import pytest

from tests.gpu_common import announce, require_gpu, to_dev
from workloads import patch_mixture as pm

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,d,G", [(3, 8, 3), (16, 8, 4), (17, 8, 4), (16, 1030, 4), (255, 33, 5), (257, 36, 7),
                                   (300, 130, 3), (1023, 7, 16), (4100, 260, 9), (16_384, 4, 40), (16_641, 12, 30),
                                   (40_000, 5, 160)])
def test_far_clusters_are_all_seeded(N, d, G):
    require_gpu()
    from paper_2606_08813_amd import hntl
    announce(f"k-means++ over {N} x {d}, {G} clusters")
    lab = (np.arange(N) * 7919) % G
    # centres 100 apart on a line, the first at 0: the greedy choice leaves no cluster out, since
    # an uncovered cluster's rows weigh >= 1e4 each, a covered one's rounding errors at most
    # 2^-22 (100 G)^2 d-independently (61 for G = 160), and 16 rows are drawn per step
    X = pm.uniform_rows(N, d, 71, lo=-0.01, hi=0.01)
    X[:, 0] += (100.0 * lab).astype(np.float32)
    ix = hntl.hntl_build(to_dev(X), G, 1, seed=5)
    ex = hntl.hntl_index_export(ix)
    np.testing.assert_array_equal(np.sort(np.diff(ex["offsets"])), np.sort(np.bincount(lab, minlength=G)))
    for g in range(G):
        members = lab[ex["perm"][ex["offsets"][g]:ex["offsets"][g + 1]]]
        assert len(set(members.tolist())) == 1
