"""GPU tests of the router's training kernels at the sizes where their tiles
end: batch rows around the reduction's row groups, layer widths that are no
multiple of its column groups, statistics over fewer rows than row runs."""
import numpy as np
import pytest

from oracle import router as orr
from tests.gpu_common import announce, require_gpu, to_dev
from workloads import patch_mixture as pm

pytestmark = pytest.mark.gpu


def small_index(hntl, G, d, seed):
    """An index of 4 G rows whose grains hold 4 rows each (arbitrary codes: only its router is used)."""
    r = 8
    X = pm.uniform_rows(4 * G, d, seed)
    st = dict(centroids=pm.uniform_rows(G, d, seed + 1), basis=pm.uniform_floats((G, r, d), seed + 2),
              offsets=4 * np.arange(G + 1, dtype=np.int64), perm=np.arange(4 * G, dtype=np.int32),
              codes=pm.uniform_floats((4 * G, r), seed + 3), eps=np.ones(4 * G, np.float32))
    return hntl.hntl_index_create(st, X)


@pytest.mark.parametrize("n,d,h1,h2,G", [(1, 8, 8, 8, 8), (63, 72, 24, 40, 16), (65, 200, 136, 56, 72),
                                         (129, 64, 128, 264, 520), (1000, 136, 72, 200, 1032)])
def test_gradients_at_odd_sizes(n, d, h1, h2, G):
    require_gpu()
    from paper_2606_08813_amd import hntl
    announce(f"router gradients, {n} rows, widths {d}-{h1}-{h2}-{G}")
    ix = small_index(hntl, G, d, 31)
    p = {k: v.astype(np.float32) for k, v in orr.init_params((d, h1, h2, G), seed=6).items()}
    X = pm.uniform_rows(n, d, 32)
    tg = pm.ints((n, 3), 33, 0, G).astype(np.int32)
    mean, std = np.zeros(d, np.float32), np.ones(d, np.float32)
    hntl.hntl_router_set(ix, p, mean, std)
    loss, g = hntl.hntl_router_grad(ix, to_dev(X), to_dev(tg))
    p64 = {k: v.astype(np.float64) for k, v in p.items()}
    s, cache = orr.forward(p64, X, mean.astype(np.float64), std.astype(np.float64), bf16=True)
    y = orr.grain_targets(tg, np.arange(G), G)
    loss_orc, ds = orr.loss_and_dlogits(s, y)
    ref = orr.backward(p64, cache, ds, bf16=True)
    assert abs(loss - loss_orc) <= 1e-4 * abs(loss_orc)
    for k in ref:
        # BF16 operands, FP32 against FP64 accumulation: the bound of the wide-layer test
        err = np.linalg.norm(g[k].astype(np.float64) - ref[k]) / max(np.linalg.norm(ref[k]), 1e-300)
        assert err < 1e-3, (k, err)


@pytest.mark.parametrize("n,d", [(1, 8), (3, 72), (64, 64), (65, 136), (1000, 200)])
def test_column_statistics(n, d):
    require_gpu()
    from paper_2606_08813_amd import hntl
    announce(f"training input statistics of {n} x {d}")
    G = 8
    ix = small_index(hntl, G, d, 41)
    X = pm.uniform_rows(n, d, 42, lo=-3.0, hi=5.0)
    X[:, 0] = 2.5  # a constant column: std 1
    tg = np.zeros((n, 1), np.int32)
    hntl.hntl_router_train(ix, to_dev(X), targets=to_dev(tg), hidden=(8, 8), epochs=1, batch=n, knn=1, lr=1e-3)
    w = hntl.hntl_router_export(ix)
    x64 = X.astype(np.float64)
    std = x64.std(0)
    std = np.where(std > 1e-12, std, 1.0)
    # FP64 sums of at most 1,000 terms, rounded once to float32 (2^-24 relative), doubled
    assert np.all(np.abs(w["mean"] - x64.mean(0)) <= 2.0 ** -23 * np.abs(x64.mean(0)) + 1e-12)
    assert np.all(np.abs(w["std"] - std) <= 2.0 ** -23 * std)
