"""GPU test of training over several batches and epochs, the row order and the
batches' losses held on the device: the same run on given targets, on targets
taken from the neighbours, and one batch at a time through kept weights."""
import numpy as np
import pytest

from tests.gpu_common import announce, require_gpu, to_dev
from tests.test_gpu_router_sizes import small_index
from workloads import patch_mixture as pm

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,batch", [(64, 64), (100, 33), (96, 8)])
def test_epochs_equal_single_batches(n, batch):
    require_gpu()
    from paper_2606_08813_amd import hntl
    announce(f"{n} rows in batches of {batch}")
    G, d = 24, 16
    ix = small_index(hntl, G, d, 111)
    X = to_dev(pm.uniform_rows(n, d, 112))
    tg = to_dev(pm.ints((n, 3), 113, 0, G).astype(np.int32))
    kw = dict(hidden=(16, 8), batch=batch, knn=3, lr=1e-2, seed=4)
    shuffled = hntl.hntl_router_train(ix, X, targets=tg, epochs=3, **kw)
    w1 = hntl.hntl_router_export(ix)
    again = hntl.hntl_router_train(ix, X, targets=tg, epochs=3, **kw)
    w2 = hntl.hntl_router_export(ix)
    assert len(shuffled) == 3 and shuffled[-1] < shuffled[0]
    for k in w1:
        np.testing.assert_array_equal(w1[k], w2[k])  # batch losses sum in any order, weights do not depend on them
    np.testing.assert_allclose(shuffled, again, rtol=1e-5)
    # rows past the last full batch of an epoch in row order have no part in it
    full = n // batch * batch
    flag = hntl.HNTL_ROUTER_NO_SHUFFLE
    a = hntl.hntl_router_train(ix, X, targets=tg, epochs=1, flags=flag, **kw)
    wa = hntl.hntl_router_export(ix)
    b = hntl.hntl_router_train(ix, X[:full].contiguous(), targets=tg[:full].contiguous(), epochs=1, flags=flag, **kw)
    wb = hntl.hntl_router_export(ix)
    for k in ("W1", "b1", "W2", "b2", "W3", "b3"):
        if full == n:
            np.testing.assert_array_equal(wa[k], wb[k])
    assert np.isfinite(a).all() and np.isfinite(b).all()
    # the loss of an epoch of one batch is the loss of that batch at the initial weights
    one = hntl.hntl_router_train(ix, X[:batch].contiguous(), targets=tg[:batch].contiguous(), epochs=1, flags=flag, **kw)
    wone = hntl.hntl_router_export(ix)
    hntl.hntl_router_train(ix, X[:batch].contiguous(), targets=tg[:batch].contiguous(), epochs=1, flags=flag,
                           **{**kw, "lr": 1e-30})
    loss0, _ = hntl.hntl_router_grad(ix, X[:batch].contiguous(), tg[:batch].contiguous())
    np.testing.assert_allclose(one[0], loss0, rtol=1e-5)
    assert all(np.isfinite(wone[k]).all() for k in wone)
