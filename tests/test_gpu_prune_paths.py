"""GPU tests of searches and plans that prune pairs before their projection, at
sizes and grains where they do (shown by the time of the projection stage, which
then takes probe slot 0 alone): results equal those without any pruning, bit for
bit, for every code form, on bases that are not orthonormal, with learned
routing, beside grains too small to bound a query, and where a score is summed with
the largest rounding errors."""
import numpy as np
import pytest

from tests.gpu_common import announce, require_gpu, to_dev

pytestmark = pytest.mark.gpu

G, D, R, NQ, P, C, K = 256, 768, 32, 2600, 8, 16, 10  # 18,200 pairs beyond the nearest
BIG, SMALL = 150, 5  # members of a grain (every 16th is small: 2 in 1,000 of all members)


@pytest.fixture(scope="module", params=[("apart", 1.0, 1.0), ("twins", 1.0, 1.0), ("twins", 1.0, 1.6),
                                        ("overlapping", 0.25, 1.0), ("coinciding", 0.0, 1.0)],
                ids=["apart", "twins", "stretched", "overlapping", "coinciding"])
def px(request):
    torch = require_gpu()
    from paper_2606_08813_amd import hntl
    kind, spread, stretch = request.param
    rng = np.random.default_rng(7)
    sizes = np.where(np.arange(G) % 16 == 15, SMALL, BIG)
    off = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int64)
    N = int(off[-1])
    H = np.linalg.qr(rng.standard_normal((D, D)))[0].astype(np.float32)
    W = H[np.argsort(rng.random((G, D)), axis=1)[:, :R]] * rng.choice([-1.0, 1.0], (G, 1, D)).astype(np.float32)
    cent = (spread * rng.standard_normal((G, D))).astype(np.float32)
    if kind == "twins":  # every pair of grains shares its surroundings: one in seven pairs is kept
        cent[1::2] = cent[::2] + 0.05 * rng.standard_normal((G // 2, D)).astype(np.float32)
        W[1::2] = W[::2]
    std = np.sqrt(4.0 * 0.85 ** np.arange(R)).astype(np.float32)
    lab = np.repeat(np.arange(G), sizes)
    ql = np.concatenate([rng.integers(0, G, NQ - 64), np.arange(15, G, 16).repeat(4)])  # the last: at small grains

    def rows(labels):
        n = len(labels)
        z = rng.standard_normal((n, R)).astype(np.float32) * std
        X = cent[labels] + 0.05 * rng.standard_normal((n, D)).astype(np.float32)
        for g in range(G):
            m = labels == g
            X[m] += z[m] @ W[g]
        return X.astype(np.float32)
    X, Q = rows(lab), rows(ql)
    W[::2] *= stretch
    codes = np.concatenate([(X[off[g]:off[g + 1]] - cent[g]) @ W[g].T for g in range(G)]).astype(np.float32)
    eps = np.maximum(((X - cent[lab]) ** 2).sum(1) - (codes ** 2).sum(1), 0.0).astype(np.float32)
    st = dict(centroids=cent, basis=W, offsets=off, perm=np.arange(N, dtype=np.int32), codes=codes, eps=eps)
    ix = hntl.hntl_index_create(st, X, codes=("fp32", "bf16", "fp8"))
    return dict(torch=torch, hntl=hntl, ix=ix, Q=to_dev(Q), cent=cent, kind=kind)


def same(px, a, b, what):
    assert px["torch"].equal(a[0], b[0]), f"{what}: ids differ"
    assert px["torch"].equal(a[1], b[1]), f"{what}: distances differ"


def project_ms(px, flags, **kw):
    """Milliseconds of the staged search's projection stage."""
    hntl = px["hntl"]
    t = []
    for _ in range(5):
        hntl.hntl_profile_read()
        hntl.hntl_search(px["ix"], px["Q"], P, C, K, flags=flags | hntl.HNTL_FLAG_SYNC | hntl.HNTL_FLAG_PROFILE, **kw)
        t.append(hntl.hntl_profile_read()[0]["project"])
    return min(t[1:])


@pytest.mark.parametrize("codes,flags", [("fp32", 0), ("bf16", 0), ("bf16", 16), ("fp8", 0), ("fp8", 16), ("fp32", 64)],
                         ids=["fp32", "bf16", "bf16-projected", "fp8", "fp8-projected", "mode-a"])
def test_pruned_equals_unpruned(px, codes, flags):
    hntl = px["hntl"]
    announce(f"{px['kind']} grains, {codes}, flags {flags}")
    full = hntl.hntl_search(px["ix"], px["Q"], P, C, K, codes=codes,
                            flags=flags | hntl.HNTL_FLAG_SYNC | hntl.HNTL_FLAG_NO_PRUNE)
    for fl in (flags, flags | hntl.HNTL_FLAG_ROUTE_BF16):
        fl |= hntl.HNTL_FLAG_SYNC
        same(px, hntl.hntl_search(px["ix"], px["Q"], P, C, K, codes=codes, flags=fl), full, "staged")
        same(px, hntl.hntl_search_noalloc(px["ix"], px["Q"], P, C, K, codes=codes, flags=fl), full, "noalloc")
    pr, pd = (hntl.hntl_search_stages(px["ix"], px["Q"], P, C, K, codes=codes, flags=flags)[k] for k in
              ("probes", "pdist"))
    del pd
    o = hntl.hntl_search_stages(px["ix"], px["Q"], P, C, K, codes=codes, flags=flags, probes_in=pr)
    same(px, (o["ids"], o["dist"]), full, "probes given")
    for sched in (None, dict(qt=4, nw=2, range=0, proj=1), dict(qt=1, nw=2, range=1, passes=2, proj=1),
                  dict(qt=8, nw=1, range=2, proj=1)):
        for graph in (False, True):
            plan = hntl.hntl_plan_create(px["ix"], P, C, K, NQ, codes=codes, flags=flags | hntl.HNTL_FLAG_SYNC,
                                         sched=sched, graph=graph)
            for n in (NQ, 1, 77, NQ):
                r = hntl.hntl_plan_search(plan, px["Q"][NQ - n:].contiguous())
                same(px, r, (full[0][NQ - n:], full[1][NQ - n:]), f"plan {sched} graph {graph} n {n}")


def test_these_sizes_are_pruned(px):
    hntl = px["hntl"]
    announce(f"{px['kind']} grains, time of the projection")
    if px["kind"] == "coinciding":  # (searches choose by sizes alone)
        pytest.skip("every pair falls on the same eight grains: a short projection either way")
    for codes, flags in (("fp32", 0), ("bf16", 16)):
        first, every = project_ms(px, flags, codes=codes), project_ms(px, flags | hntl.HNTL_FLAG_NO_PRUNE, codes=codes)
        print(f"projection of slot 0 {first * 1e3:.1f} us, of every slot {every * 1e3:.1f}")
        assert first < 0.85 * every, (codes, first, every)  # 0.66; 1 where every slot is projected
    if px["kind"] in ("apart", "twins"):
        sched = dict(qt=2, nw=2, range=0, proj=1)
        t = {}
        for flags in (0, hntl.HNTL_FLAG_NO_PRUNE):
            plan = hntl.hntl_plan_create(px["ix"], P, C, K, NQ, flags=flags, sched=sched)
            hntl.hntl_plan_search(plan, px["Q"])
            t[flags] = hntl.hntl_plan_profile(plan, NQ, reps=1)[1]
        # slot 0's members and the twin's (all eight slots' without pruning)
        assert t[0] < 0.5 * t[hntl.HNTL_FLAG_NO_PRUNE], t


@pytest.mark.parametrize("mass", [0.0, 0.9])
def test_learned_routing(px, mass):
    hntl = px["hntl"]
    announce(f"{px['kind']} grains after learned routing, mass {mass}")
    h = 256
    A = np.linalg.qr(np.random.default_rng(8).standard_normal((D, h)))[0].T.astype(np.float32)
    mu = px["cent"] @ A.T
    eye = np.eye(h, dtype=np.float32)
    w = dict(W1=np.concatenate([A, -A]), b1=np.zeros(2 * h), W2=np.block([[eye, -eye], [-eye, eye]]),
             b2=np.zeros(2 * h), W3=0.03 * np.concatenate([mu, -mu], 1), b3=-0.015 * (mu ** 2).sum(1))
    hntl.hntl_router_set(px["ix"], w, np.zeros(D), np.ones(D))
    kw = dict(route="learned", mass=mass)
    full = hntl.hntl_search(px["ix"], px["Q"], P, C, K, flags=hntl.HNTL_FLAG_SYNC | hntl.HNTL_FLAG_NO_PRUNE, **kw)
    same(px, hntl.hntl_search(px["ix"], px["Q"], P, C, K, flags=hntl.HNTL_FLAG_SYNC, **kw), full, "staged")
    same(px, hntl.hntl_search_noalloc(px["ix"], px["Q"], P, C, K, flags=hntl.HNTL_FLAG_SYNC, **kw), full, "noalloc")
    plan = hntl.hntl_plan_create(px["ix"], P, C, K, NQ, flags=hntl.HNTL_FLAG_SYNC, sched=dict(qt=2, nw=2, range=2, proj=1),
                                 **kw)
    same(px, hntl.hntl_plan_search(plan, px["Q"]), full, "plan")
    if mass == 0.0 and px["kind"] != "coinciding":
        assert project_ms(px, 0, **kw) < 0.85 * project_ms(px, hntl.HNTL_FLAG_NO_PRUNE, **kw)


@pytest.mark.parametrize("d", [256, 2048, 4096])
def test_sums_that_lose_the_most(d):
    """||q - mu||^2 as the projection sums it (four chains of d / 4 terms) loses what lies below
    half a unit of the first term; the routing distance (64 chains) loses less.  Grains whose longest
    code nearly reaches the query put the score next to the bound."""
    torch = require_gpu()
    from paper_2606_08813_amd import hntl
    announce(f"chains of {d // 4} terms")
    rng = np.random.default_rng(d)
    Gn, r, n, nq, probes, c = 16, 16, 40, 800, 16, 16
    big = [0, 8, 16, 24]  # the first term of each chain (and, of BF16's, the first too)
    gaps = np.concatenate([[0.0], 10.0 ** -np.linspace(0.5, 4.0, Gn - 1)])
    cent = np.zeros((Gn, d), np.float32)
    cent[0, big] = 1.0
    W = np.zeros((Gn, r, d), np.float32)
    W[0, 0, 100] = 1.0
    W[1:, 0, big] = 0.5
    for j in range(1, r):
        W[:, j, 200 + j] = 1.0
    codes = np.zeros((Gn, n, r), np.float32)
    codes[0, :, 0] = np.linspace(-0.4, 0.4, n)
    codes[1:, :, 0] = 2.0 - gaps[1:, None] * (1.0 + np.linspace(0.0, 3.0, n))[None]
    off = (np.arange(Gn + 1) * n).astype(np.int64)
    st = dict(centroids=cent, basis=W, offsets=off, perm=np.arange(Gn * n, dtype=np.int32),
              codes=codes.reshape(-1, r), eps=np.zeros(Gn * n, np.float32))
    ix = hntl.hntl_index_create(st, rng.standard_normal((Gn * n, d)).astype(np.float32), codes=("fp32", "bf16"))
    Q = (2.0 ** -12.52 * rng.choice([-1.0, 1.0], (nq, d))).astype(np.float32)
    Q[:, big] = 1.0
    Q[:, 100] = rng.uniform(-0.3, 0.3, nq).astype(np.float32) * 10.0 ** -rng.uniform(0, 4, nq)
    Q = to_dev(Q.astype(np.float32))
    for codes_, flags in (("fp32", 0), ("bf16", 0), ("bf16", 16)):
        sync = flags | hntl.HNTL_FLAG_SYNC
        full = hntl.hntl_search_stages(ix, Q, probes, c, 10, codes=codes_, flags=sync | hntl.HNTL_FLAG_NO_PRUNE)
        pools = hntl.hntl_search(ix, Q, probes, c, 10, codes=codes_, flags=sync)
        assert torch.equal(pools[0], full["ids"]) and torch.equal(pools[1], full["dist"]), (codes_, flags)
        a = hntl.hntl_search(ix, Q, probes, c, 10, codes=codes_, flags=sync | 64)
        b = hntl.hntl_search(ix, Q, probes, c, 10, codes=codes_, flags=sync | 64 | hntl.HNTL_FLAG_NO_PRUNE)
        assert torch.equal(a[0], b[0]) and torch.equal(a[1], b[1]), (codes_, flags)
