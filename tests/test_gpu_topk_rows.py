"""GPU tests of the selection of the P best grains of a row at the row lengths
where its registers end (64 values a lane and chunk, 16 / 32 / 64 / 128 chunks)
and with more entries inside the re-score window than a wave can hold."""
import numpy as np
import pytest

from oracle import router as orr, search as osr
from tests import parity
from tests.gpu_common import announce, centroid_dist_fn, require_gpu, to_dev
from tests.test_gpu_router_sizes import small_index
from tests.test_gpu_tiles import plain_index
from workloads import patch_mixture as pm

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("G,P,copies", [(1, 1, 0), (63, 48, 0), (64, 48, 0), (65, 1, 30), (1024, 8, 70), (1025, 48, 0),
                                        (2048, 16, 100), (2049, 16, 40), (4096, 48, 0), (4097, 8, 65), (8191, 48, 30),
                                        (8192, 8, 200), (8193, 8, 200), (8193, 48, 0)])
@pytest.mark.parametrize("nq", [3, 70])
def test_nearest_grains(G, P, copies, nq):
    require_gpu()
    from paper_2606_08813_amd import hntl
    announce(f"{P} of {G} grains for {nq} queries, {copies} equal centroids")
    d = 16
    cent = pm.uniform_rows(G, d, 51)
    Q = pm.uniform_rows(nq, d, 52)
    if copies:  # equal centroids spread over the row, close to every second query: the lower ids win
        at = np.linspace(0, G - 1, copies).astype(np.int64)
        cent[at] = cent[at[0]]
        Q[::2] = cent[at[0]] + 1e-3 * Q[::2]
    ix = plain_index(hntl, cent, cent, r=8)
    o = hntl.hntl_search_stages(ix, to_dev(Q), P, 8, 1)
    ref, ref_d = osr.route(Q, cent, P)
    parity.check_lists(o["probes"].cpu().numpy(), o["pdist"].cpu().numpy(), ref, ref_d, centroid_dist_fn(cent, Q),
                       what="probes")
    if copies > P:
        np.testing.assert_array_equal(np.sort(o["probes"].cpu().numpy()[0]), np.sort(at[:P]))


@pytest.mark.parametrize("G,P", [(8, 1), (72, 48), (1024, 8), (1032, 16), (2048, 48), (4104, 8), (8192, 16), (8200, 16)])
def test_best_scores(G, P):
    require_gpu()
    from paper_2606_08813_amd import hntl
    announce(f"{P} best of {G} scores")
    nq, d, h = 70, 16, 16
    ix = small_index(hntl, G, d, 61)
    p = {k: v.astype(np.float32) for k, v in orr.init_params((d, h, h, G), seed=7).items()}
    p["W3"] = p["W3"] * 8.0
    p["b3"] = p["b3"] + pm.ints((G,), 62, 0, 8).astype(np.float32)  # peaked: the budget ends inside the list
    hntl.hntl_router_set(ix, p, np.zeros(d, np.float32), np.ones(d, np.float32))
    Q = to_dev(pm.uniform_rows(nq, d, 63))
    s = hntl.hntl_router_forward(ix, Q).cpu().numpy()
    ref = np.lexsort((np.broadcast_to(np.arange(G), s.shape), -s), axis=1)[:, :P]
    got = hntl.hntl_search_stages(ix, Q, P, 8, 1, route="learned")["probes"].cpu().numpy()
    np.testing.assert_array_equal(got, ref)
    mass = 0.02
    cut = hntl.hntl_search_stages(ix, Q, P, 8, 1, route="learned", mass=mass)["probes"].cpu().numpy()
    # rows whose cumulative probability passes the budget by more than float32 sums
    # of G terms can move it (G 2^-24 < 5e-4 relative; the terms are all positive)
    e = np.exp(s.astype(np.float64) - s.max(axis=1, keepdims=True))
    c = np.cumsum(np.take_along_axis(e, ref, 1), axis=1) / e.sum(axis=1, keepdims=True)
    clear = (np.abs(c - mass) > 1e-3 * mass).all(axis=1)
    assert clear.sum() >= nq // 2
    np.testing.assert_array_equal(cut[clear], orr.mass_cut(s, ref, mass)[clear])
