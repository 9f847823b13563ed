"""GPU tests of the small BF16 products behind the router at the sizes where
their 64 x 64 x 64 tiles end: scores of a few rows, gradients over odd batches."""
import numpy as np
import pytest

from oracle import router as orr
from tests.gpu_common import announce, require_gpu, to_dev
from tests.test_gpu_router_sizes import small_index
from tests.test_gpu_tiles import plain_index
from workloads import patch_mixture as pm

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,d,h1,h2,G", [(1, 8, 8, 8, 8), (63, 56, 64, 72, 128), (64, 64, 64, 64, 64),
                                         (65, 72, 128, 120, 200), (257, 320, 264, 512, 136), (512, 768, 192, 256, 1032)])
def test_scores_and_gradients(n, d, h1, h2, G):
    require_gpu()
    from paper_2606_08813_amd import hntl
    announce(f"router products, {n} rows, widths {d}-{h1}-{h2}-{G}")
    ix = small_index(hntl, G, d, 91)
    p = {k: v.astype(np.float32) for k, v in orr.init_params((d, h1, h2, G), seed=9).items()}
    X = pm.uniform_rows(n, d, 92)
    tg = pm.ints((n, 2), 93, 0, G).astype(np.int32)
    mean, std = np.zeros(d, np.float32), np.ones(d, np.float32)
    hntl.hntl_router_set(ix, p, mean, std)
    p64 = {k: v.astype(np.float64) for k, v in p.items()}
    s, cache = orr.forward(p64, X, mean.astype(np.float64), std.astype(np.float64), bf16=True)
    got = hntl.hntl_router_forward(ix, to_dev(X)).cpu().numpy().astype(np.float64)
    # FP32 against FP64 accumulation; a hidden value whose rounding to BF16 turns over moves by 2^-8 of itself
    assert np.linalg.norm(got - s) <= 1e-3 * np.linalg.norm(s)
    loss, g = hntl.hntl_router_grad(ix, to_dev(X), to_dev(tg))
    y = orr.grain_targets(tg, np.arange(G), G)
    loss_orc, ds = orr.loss_and_dlogits(s, y)
    ref = orr.backward(p64, cache, ds, bf16=True)
    assert abs(loss - loss_orc) <= 1e-4 * abs(loss_orc)
    for k in ref:
        err = np.linalg.norm(g[k].astype(np.float64) - ref[k]) / max(np.linalg.norm(ref[k]), 1e-300)
        assert err < 1e-3, (k, err)  # the bound of the wide-layer test


@pytest.mark.parametrize("nq,G", [(4160, 4101), (4100, 4099), (5000, 4225)])
@pytest.mark.parametrize("flag", ["HNTL_FLAG_ROUTE_BF16", "HNTL_FLAG_ROUTE_BF16X3"])
def test_large_tiles_at_odd_column_counts(nq, G, flag):
    """256 x 256 tiles whose rows of results start at any 4-byte address and whose last columns are no whole run."""
    torch = require_gpu()
    from paper_2606_08813_amd import hntl
    announce(f"{flag}: {nq} x {G}")
    d, P = 64, 4
    cent = pm.uniform_rows(G, d, 94)
    Q = pm.uniform_rows(nq, d, 95)
    ix = plain_index(hntl, cent, cent, r=8)
    o = hntl.hntl_search_stages(ix, to_dev(Q), P, 8, 1, flags=hntl.HNTL_FLAG_SYNC | getattr(hntl, flag))
    full = hntl.hntl_search_stages(ix, to_dev(Q), P, 8, 1)
    # the re-scored nearest grains do not depend on the form of the product
    assert torch.equal(o["probes"], full["probes"])
    assert torch.equal(o["pdist"], full["pdist"])
