"""GPU tests of the pruning before projection: batches large enough to take it
must give the results of a search without any pruning, bit for bit, whether the
grains lie far apart (nearly every pair goes), overlap (some do) or coincide
(none do), for every code form, on bases that are not orthonormal, with
learned routing (the distances computed by the pruning itself) and for batch
sizes below a plan's."""
import numpy as np
import pytest

from tests.gpu_common import announce, require_gpu, to_dev
from workloads import patch_mixture as pm

pytestmark = pytest.mark.gpu

N, G, D, R, NQ, P, C, K = 20_001, 513, 768, 48, 520, 8, 40, 10  # 513 x 48 x 768 x 4 B of bases: 76 MB


@pytest.fixture(scope="module", params=[(1.0, 1.0), (0.12, 1.0), (0.0, 1.0), (0.12, 1.6)],
                ids=["apart", "overlapping", "coinciding", "stretched-bases"])
def px(request):
    torch = require_gpu()
    from paper_2606_08813_amd import hntl
    spread, stretch = request.param
    rng = np.random.default_rng(71)
    H = np.linalg.qr(rng.standard_normal((D, D)))[0].astype(np.float32)
    lab = np.sort(rng.integers(0, G - 1, N))  # the last grain is empty
    lab[:64] = 0
    off = np.searchsorted(lab, np.arange(G + 1)).astype(np.int64)
    off[-1] = N
    W = H[np.argsort(rng.random((G, D)), axis=1)[:, :R]] * rng.choice([-1.0, 1.0], (G, 1, D)).astype(np.float32)
    cent = (spread * rng.standard_normal((G, D))).astype(np.float32)
    std = np.sqrt(4.0 * 0.85 ** np.arange(R)).astype(np.float32)
    X = (0.05 * rng.standard_normal((N, D))).astype(np.float32)
    Q = (0.05 * rng.standard_normal((NQ, D))).astype(np.float32)
    ql = rng.integers(0, G - 1, NQ)
    for g in range(G):
        n, m = int(off[g + 1] - off[g]), int((ql == g).sum())
        X[off[g]:off[g + 1]] += cent[g] + (rng.standard_normal((n, R)).astype(np.float32) * std) @ W[g]
        Q[ql == g] += cent[g] + (rng.standard_normal((m, R)).astype(np.float32) * std) @ W[g]
    W[::2] *= stretch
    codes = np.concatenate([(X[off[g]:off[g + 1]] - cent[g]) @ W[g].T for g in range(G)]).astype(np.float32)
    eps = ((X - cent[lab]) ** 2).sum(1) - (codes ** 2).sum(1)
    st = dict(centroids=cent, basis=W, offsets=off, perm=np.arange(N, dtype=np.int32), codes=codes,
              eps=np.maximum(eps, 0.0).astype(np.float32))
    ix = hntl.hntl_index_create(st, X, codes=("fp32", "bf16", "fp8"))
    return dict(torch=torch, hntl=hntl, ix=ix, Q=to_dev(Q), X=X, cent=cent)


def same(px, a, b, what):
    assert px["torch"].equal(a[0], b[0]), f"{what}: ids differ"
    assert px["torch"].equal(a[1], b[1]), f"{what}: distances differ"


@pytest.mark.parametrize("codes,flags", [("fp32", 0), ("bf16", 16), ("fp8", 0), ("fp32", 64)],
                         ids=["fp32", "bf16-projected", "fp8", "mode-a"])
def test_pruned_equals_unpruned(px, codes, flags):
    hntl = px["hntl"]
    announce(f"pruning before projection, {codes}, flags {flags}")
    fl = flags | hntl.HNTL_FLAG_SYNC | hntl.HNTL_FLAG_ROUTE_BF16
    full = hntl.hntl_search(px["ix"], px["Q"], P, C, K, codes=codes, flags=fl | hntl.HNTL_FLAG_NO_PRUNE)
    same(px, hntl.hntl_search(px["ix"], px["Q"], P, C, K, codes=codes, flags=fl), full, "staged")
    same(px, hntl.hntl_search_noalloc(px["ix"], px["Q"], P, C, K, codes=codes, flags=fl), full, "noalloc")
    for sched in (dict(qt=4, nw=2, range=0, proj=1), dict(qt=1, nw=2, range=1, passes=2, proj=1),
                  dict(qt=8, nw=1, range=4, proj=1)):
        for graph in (False, True):
            plan = hntl.hntl_plan_create(px["ix"], P, C, K, NQ, codes=codes, flags=fl, sched=sched, graph=graph)
            for n in (NQ, 1, 77, NQ):
                r = hntl.hntl_plan_search(plan, px["Q"][:n].contiguous())
                same(px, r, (full[0][:n], full[1][:n]), f"plan {sched} graph {graph} n {n}")


@pytest.mark.parametrize("mass", [0.0, 0.9])
def test_learned_routing(px, mass):
    hntl = px["hntl"]
    announce(f"pruning after learned routing, mass {mass}")
    # the router needs a multiple of 8 grains: the same index without its last (empty) grain
    st = hntl.hntl_index_export(px["ix"])
    st = dict(st, centroids=st["centroids"][:G - 1].copy(), basis=st["basis"][:G - 1].copy(),
              offsets=st["offsets"][:G].copy())
    ix = hntl.hntl_index_create(st, px["X"])
    h = 512
    A = np.linalg.qr(np.random.default_rng(72).standard_normal((D, h)))[0].T.astype(np.float32)
    mu = px["cent"][:G - 1] @ A.T
    eye = np.eye(h, dtype=np.float32)
    w = dict(W1=np.concatenate([A, -A]), b1=np.zeros(2 * h), W2=np.block([[eye, -eye], [-eye, eye]]),
             b2=np.zeros(2 * h), W3=0.03 * np.concatenate([mu, -mu], 1), b3=-0.015 * (mu ** 2).sum(1))
    hntl.hntl_router_set(ix, w, np.zeros(D), np.ones(D))
    fl = hntl.HNTL_FLAG_SYNC
    full = hntl.hntl_search(ix, px["Q"], P, C, K, flags=fl | hntl.HNTL_FLAG_NO_PRUNE, route="learned", mass=mass)
    same(px, hntl.hntl_search(ix, px["Q"], P, C, K, flags=fl, route="learned", mass=mass), full, "staged")
    plan = hntl.hntl_plan_create(ix, P, C, K, NQ, flags=fl, sched=dict(qt=2, nw=2, range=2, proj=1),
                                 route="learned", mass=mass)
    same(px, hntl.hntl_plan_search(plan, px["Q"]), full, "plan")
