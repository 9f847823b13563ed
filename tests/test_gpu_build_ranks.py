"""GPU build over the ranks and row lengths where the orthonormalisation changes
its form or its triangle ends: r + 16 or 2 r columns, at most d of them."""
import pytest

from tests.gpu_common import announce, require_gpu, to_dev
from tests.test_gpu_build import _check_invariants
from workloads import patch_mixture as pm

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,d,G,r", [(400, 1, 3, 1), (500, 20, 4, 8), (900, 33, 5, 16), (900, 260, 5, 17), (700, 64, 4, 24),
                                     (1500, 96, 4, 33), (1500, 130, 4, 48), (1500, 100, 3, 50), (2000, 300, 3, 64)])
def test_orthonormal_bases(N, d, G, r):
    require_gpu()
    from paper_2606_08813_amd import hntl
    announce(f"local PCA of {N} x {d}, {G} grains, rank {r}")
    X = pm.uniform_rows(N, d, 81)
    ix = hntl.hntl_build(to_dev(X), G, r, seed=3)
    _check_invariants(X, hntl.hntl_index_export(ix), hntl.hntl_index_captured(ix))
