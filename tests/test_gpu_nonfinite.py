"""GPU tests of query rows that hold NaN or infinity in calls that do not check
for them (asynchronous searches, plans, neighbour searches): such a row names no
grain twice, and every other row of the batch gets what it gets alone."""
import numpy as np
import pytest

from tests.gpu_common import announce, require_gpu, to_dev
from workloads import patch_mixture as pm

pytestmark = pytest.mark.gpu

R, P, C, K = 16, 4, 32, 8


def index(hntl, d, sizes, seed=5, spread=1.0):
    """Grains of the given sizes around normal centres, the last one included."""
    rng = np.random.default_rng(seed)
    G, off = len(sizes), np.concatenate([[0], np.cumsum(sizes)]).astype(np.int64)
    N = int(off[-1])
    cent = (spread * rng.standard_normal((G, d))).astype(np.float32)
    W = np.stack([np.linalg.qr(rng.standard_normal((d, R)))[0].T for _ in range(G)]).astype(np.float32)
    z = rng.standard_normal((N, R)).astype(np.float32)
    lab = np.repeat(np.arange(G), sizes)
    X = cent[lab] + np.einsum("nr,nrd->nd", z, W[lab]).astype(np.float32)
    st = dict(centroids=cent, basis=W, offsets=off, perm=np.arange(N, dtype=np.int32), codes=z,
              eps=np.full(N, 0.01, np.float32))
    return hntl.hntl_index_create(st, X), X


def spoil(Q, rows, value):
    B = Q.clone()
    for r in rows:
        B[r, r % Q.shape[1]] = value
    return B


@pytest.mark.parametrize("value", [float("nan"), float("inf")], ids=["nan", "inf"])
@pytest.mark.parametrize("nq", [3, 16, 17, 40])  # direct differences up to 16 rows, products above
def test_probes_are_different_grains(nq, value):
    require_gpu()
    from paper_2606_08813_amd import hntl
    announce(f"probes of {nq} rows, one of them {value}")
    ix, X = index(hntl, 32, [50] * 11)
    Q = to_dev(X[::13][:nq].copy())
    bad = spoil(Q, [1], value)
    o = hntl.hntl_search_stages(ix, bad, P, C, K, flags=0)
    ref = hntl.hntl_search_stages(ix, Q, P, C, K, flags=0)
    pr = o["probes"].cpu().numpy()
    for row in pr:
        valid = row[row >= 0]
        assert len(set(valid.tolist())) == len(valid) and (valid < 11).all()
    if nq <= 16 and value != value:  # no distance is a number: no probes, no results
        assert (pr[1] == -1).all() and (o["pdist"][1].cpu().numpy() == np.inf).all()
        assert (o["ids"][1] == -1).all() and (o["dist"][1].cpu().numpy() == np.inf).all()
    keep = [i for i in range(nq) if i != 1]
    for k in ("probes", "pdist", "zq", "epsq", "pool_ids", "pool_D", "ids", "dist"):
        np.testing.assert_array_equal(o[k].cpu().numpy()[keep], ref[k].cpu().numpy()[keep], err_msg=k)


def test_centroid_that_is_not_a_number():
    require_gpu()
    from paper_2606_08813_amd import hntl
    announce("six probes of six grains, one centroid NaN")
    ix, X = index(hntl, 32, [50] * 6)
    st = hntl.hntl_index_export(ix)
    st["centroids"][2, 5] = np.nan
    nx = hntl.hntl_index_create(st, X)
    o = hntl.hntl_search_stages(nx, to_dev(X[::40].copy()), 6, C, K, flags=0)
    pr, pd = o["probes"].cpu().numpy(), o["pdist"].cpu().numpy()
    assert (np.sort(pr[:, :5], 1) == [0, 1, 3, 4, 5]).all() and (pr[:, 5] == -1).all()
    assert np.isfinite(pd[:, :5]).all() and (pd[:, 5] == np.inf).all()


@pytest.mark.parametrize("value", [float("nan"), float("inf")], ids=["nan", "inf"])
@pytest.mark.parametrize("sched", [None, dict(qt=1, nw=1, range=1), dict(qt=1, nw=2, range=2, passes=2, proj=1)],
                         ids=["default", "range1", "proj"])
def test_small_plans_over_split_grains(sched, value):
    torch = require_gpu()
    from paper_2606_08813_amd import hntl
    announce(f"plans of up to 16 rows over grains of block ranges, {sched}, {value}")
    # the last grain has more block ranges than the others together
    ix, X = index(hntl, 32, [70, 20, 130, 65, 10, 5000])
    for max_nq in (1, 2, 7, 16):
        Q = to_dev(X[::97][:max_nq].copy())
        rows = sorted({0, max_nq // 2})
        bad = spoil(Q, rows, value)
        plan = hntl.hntl_plan_create(ix, P, C, K, max_nq, sched=sched)
        want = [t.clone() for t in hntl.hntl_plan_search(plan, Q)]
        got = hntl.hntl_plan_search(plan, bad)
        torch.cuda.synchronize()
        keep = [i for i in range(max_nq) if i not in rows]
        for a, b in zip(got, want):
            assert torch.equal(a[keep], b[keep])
        if value != value:
            assert (got[0][rows] == -1).all()
        again = hntl.hntl_plan_search(plan, Q)
        assert torch.equal(again[0], want[0]) and torch.equal(again[1], want[1])
        assert hntl.hntl_plan_info_get(plan)["wait_errors"] == 0


@pytest.mark.parametrize("value", [float("nan"), float("inf"), -float("inf")], ids=["nan", "inf", "-inf"])
def test_batches_that_prune_pairs(value):
    torch = require_gpu()
    from paper_2606_08813_amd import hntl
    announce(f"pruning batches with rows of {value}")
    nq, probes = 1800, 8  # 12,600 pairs beyond the nearest: searches and plans prune before projection
    ix, X = index(hntl, 64, [300] * 40, spread=4.0)
    Q = to_dev(X[np.random.default_rng(3).integers(0, len(X), nq)] + 0.01)
    rows = [0, 5, 700, nq - 1]
    bad = spoil(Q, rows, value)
    keep = [i for i in range(nq) if i not in rows]
    want = hntl.hntl_search(ix, Q, probes, C, K, flags=hntl.HNTL_FLAG_SYNC)
    runs = {"staged": hntl.hntl_search(ix, bad, probes, C, K)}
    for flags in (0, hntl.HNTL_FLAG_ROUTE_BF16):
        plan = hntl.hntl_plan_create(ix, probes, C, K, nq, flags=flags)
        runs[f"plan {flags}"] = hntl.hntl_plan_search(plan, bad)
    torch.cuda.synchronize()
    for what, r in runs.items():
        assert torch.equal(r[0][keep], want[0][keep]) and torch.equal(r[1][keep], want[1][keep]), what


@pytest.mark.parametrize("value", [float("nan"), float("inf")], ids=["nan", "inf"])
@pytest.mark.parametrize("nq,d", [(5, 32), (70, 32), (200, 64), (20, 33)])
def test_neighbours_of_the_other_rows(nq, d, value):
    torch = require_gpu()
    from paper_2606_08813_amd import hntl
    announce(f"neighbours of {nq} x {d} rows, one of them {value}")
    X = pm.uniform_rows(3000, d, 11)
    st = dict(centroids=X[:1].copy(), basis=pm.uniform_floats((1, 8, d), 3), offsets=np.array([0, 3000], np.int64),
              perm=np.arange(3000, dtype=np.int32), codes=pm.uniform_floats((3000, 8), 4), eps=np.ones(3000, np.float32))
    ix = hntl.hntl_index_create(st, X)
    Q = to_dev(pm.uniform_rows(nq, d, 12))
    want = hntl.hntl_knn(ix, Q, 10)
    got = hntl.hntl_knn(ix, spoil(Q, [3], value), 10)
    keep = [i for i in range(nq) if i != 3]
    assert torch.equal(got[0][keep], want[0][keep]) and torch.equal(got[1][keep], want[1][keep])
