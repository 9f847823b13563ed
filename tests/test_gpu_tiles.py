"""GPU tests of the FP32 distance tiles (centroid routing and brute-force
neighbours) at the sizes where a tile, a depth chunk or a column range ends,
against float64 distances."""
import numpy as np
import pytest

from oracle import brute, search as osr
from tests import parity
from tests.gpu_common import announce, centroid_dist_fn, exact_dist_fn, require_gpu, to_dev
from workloads import patch_mixture as pm

pytestmark = pytest.mark.gpu


def plain_index(hntl, X, cent, r=8):
    """An index with one grain per centroid, rows dealt out evenly (its codes are not used here)."""
    N, d = X.shape
    G = cent.shape[0]
    off = (np.arange(G + 1, dtype=np.int64) * N) // G
    st = dict(centroids=cent, basis=pm.uniform_floats((G, r, d), 3), offsets=off, perm=np.arange(N, dtype=np.int32),
              codes=pm.uniform_floats((N, r), 4), eps=np.ones(N, np.float32))
    return hntl.hntl_index_create(st, X)


@pytest.mark.parametrize("nq,N,d,k", [
    (1, 1, 8, 1), (1, 31, 12, 10), (16, 127, 32, 16), (17, 129, 36, 3), (15, 5000, 4, 16), (64, 1000, 100, 10),
    (65, 2049, 64, 10), (128, 3000, 28, 16), (129, 1024, 768, 10), (193, 4099, 96, 7), (300, 20_011, 40, 16),
    (20, 3000, 33, 5), (70, 500, 7, 10)])  # the last two: rows without 16-byte alignment
def test_neighbours_at_tile_edges(nq, N, d, k):
    require_gpu()
    from paper_2606_08813_amd import hntl
    announce(f"{k} nearest of {N} x {d} for {nq} queries")
    k = min(k, N)
    X = pm.uniform_rows(N, d, 11)
    if N > 200:
        X[100:140] = X[99]  # exact ties, more than a list holds: the lower ids win
    Q = pm.uniform_rows(nq, d, 12)
    Q[0] = X[min(99, N - 1)]
    ix = plain_index(hntl, X, X[:1].copy(), r=min(8, d))
    ids, dist = hntl.hntl_knn(ix, to_dev(Q), k)
    ref_ids, ref_dist = brute.knn(X, Q, k)
    # routing expansions of values near 1 lose up to 1e-6 absolute next to a distance of 0
    parity.check_lists(ids.cpu().numpy(), dist.cpu().numpy(), ref_ids, ref_dist, exact_dist_fn(X, Q), what="knn")


@pytest.mark.parametrize("nq,G,d,P", [(17, 9, 8, 3), (63, 65, 36, 5), (64, 64, 64, 4), (65, 63, 100, 16),
                                      (200, 130, 4, 8), (4100, 2056, 196, 3), (8200, 2056, 228, 3), (130, 70, 33, 4),
                                      (17, 9, 192, 3), (63, 65, 204, 5), (65, 63, 768, 16), (129, 130, 256, 8)])
def test_probes_at_tile_edges(nq, G, d, P):
    require_gpu()
    from paper_2606_08813_amd import hntl
    announce(f"FP32 routing of {nq} queries over {G} x {d} centroids")
    cent = pm.uniform_rows(G, d, 21)
    Q = pm.uniform_rows(nq, d, 22)
    ix = plain_index(hntl, cent, cent, r=min(8, d))
    o = hntl.hntl_search_stages(ix, to_dev(Q), P, 8, 1)
    ref, ref_d = osr.route(Q, cent, P)
    parity.check_lists(o["probes"].cpu().numpy(), o["pdist"].cpu().numpy(), ref, ref_d, centroid_dist_fn(cent, Q),
                       what="probes")
