"""GPU tests that training takes its rows and their targets batch by batch in the
order it states: against the same epochs driven one batch at a time from here
(gradients of each batch at the current weights, Adam on the host), in row order
and shuffled, and targets from the neighbours against the same targets given."""
import numpy as np
import pytest

from tests.gpu_common import announce, require_gpu, to_dev
from tests.test_gpu_router_sizes import small_index
from workloads import patch_mixture as pm

pytestmark = pytest.mark.gpu

NAMES = ("W1", "b1", "W2", "b2", "W3", "b3")
M64 = (1 << 64) - 1


def splitmix(x):
    x = (x + 0x9E3779B97F4A7C15) & M64
    x = ((x ^ (x >> 30)) * 0xBF58476D1CE4E5B9) & M64
    x = ((x ^ (x >> 27)) * 0x94D049BB133111EB) & M64
    return x ^ (x >> 31)


def uni(seed, stream, i):
    return (splitmix((splitmix(seed ^ ((stream * 0xD1B54A32D192ED03) & M64)) + i) & M64) >> 11) / 9007199254740992.0


def shuffle(order, seed, epoch):
    for i in range(len(order) - 1, 0, -1):
        j = min(int(uni(seed, 100 + epoch, i) * (i + 1)), i)
        order[i], order[j] = order[j], order[i]


def epochs_from_here(hntl, ix, w0, X, tg, batch, epochs, lr, seed, shuffled):
    """Weights and mean losses after the epochs."""
    w = {k: w0[k].copy() for k in NAMES}
    m = {k: np.zeros_like(w[k]) for k in NAMES}
    v = {k: np.zeros_like(w[k]) for k in NAMES}
    order, losses, t = list(range(len(X))), [], 0
    for ep in range(epochs):
        if shuffled:
            shuffle(order, seed, ep)
        total = []
        for b in range(len(X) // batch):
            rows = order[b * batch:(b + 1) * batch]
            hntl.hntl_router_set(ix, w, w0["mean"], w0["std"])
            loss, g = hntl.hntl_router_grad(ix, to_dev(X[rows]), to_dev(tg[rows]))
            total.append(loss)
            t += 1
            for k in NAMES:
                gk = g[k].astype(np.float64)
                m[k] = (0.9 * m[k] + (1 - 0.9) * gk).astype(np.float32)
                v[k] = (0.999 * v[k] + (1 - 0.999) * gk * gk).astype(np.float32)
                step = lr * (m[k] / (1 - 0.9 ** t)) / (np.sqrt(v[k] / (1 - 0.999 ** t)) + 1e-8)
                w[k] = (w[k] - step).astype(np.float32)
        losses.append(np.mean(total))
    return w, losses


@pytest.mark.parametrize("n,batch,epochs,shuffled", [(64, 16, 1, False), (100, 33, 1, False), (96, 24, 2, True),
                                                     (70, 16, 2, True), (40, 40, 2, False)])
def test_epochs_equal_batches_driven_from_here(n, batch, epochs, shuffled):
    require_gpu()
    from paper_2606_08813_amd import hntl
    announce(f"{epochs} epochs of {n} rows in batches of {batch}, shuffled {shuffled}")
    G, d, lr, seed = 24, 16, 1e-2, 9
    ix = small_index(hntl, G, d, 121)
    X = pm.uniform_rows(n, d, 122)
    tg = pm.ints((n, 3), 123, 0, G).astype(np.int32)
    flags = 0 if shuffled else hntl.HNTL_ROUTER_NO_SHUFFLE
    kw = dict(targets=to_dev(tg), hidden=(16, 8), batch=batch, knn=3, seed=seed, flags=flags)
    hntl.hntl_router_train(ix, to_dev(X), epochs=1, lr=1e-30, **kw)
    w0 = hntl.hntl_router_export(ix)  # the initial weights
    losses = hntl.hntl_router_train(ix, to_dev(X), epochs=epochs, lr=lr, **kw)
    got = hntl.hntl_router_export(ix)
    want, ref_losses = epochs_from_here(hntl, ix, w0, X, tg, batch, epochs, lr, seed, shuffled)
    # The steps are of size lr whatever the gradients' size; both sides take them from the same
    # gradient kernels, at weights that a rounding of the update may set apart by 2^-23 of them: a few
    # BF16 operands then round the other way, which moves a step by a small part of lr and can turn
    # it only where a gradient is next to nothing.
    for k in NAMES:
        diff = np.abs(got[k].astype(np.float64) - want[k])
        moved = np.abs(got[k].astype(np.float64) - w0[k])
        assert moved.mean() > 0.2 * lr, k
        assert diff.mean() < 0.02 * lr and (diff > 0.1 * lr).mean() < 0.02, (k, diff.mean() / lr, diff.max() / lr)
    np.testing.assert_allclose(losses, ref_losses, rtol=1e-4)
    # another order of the batch's targets is another run
    other, _ = epochs_from_here(hntl, ix, w0, X, np.roll(tg, 1, 0), batch, epochs, lr, seed, shuffled)
    assert np.abs(got["W3"] - other["W3"]).mean() > 0.1 * lr


@pytest.mark.parametrize("shuffled", [False, True])
def test_neighbour_targets_equal_the_same_targets_given(shuffled):
    require_gpu()
    from paper_2606_08813_amd import hntl
    announce(f"targets from the neighbours, shuffled {shuffled}")
    G, d, n, kt = 24, 16, 90, 5
    ix = small_index(hntl, G, d, 131)
    X = to_dev(pm.uniform_rows(n, d, 132))
    ids, _ = hntl.hntl_knn(ix, X, kt)
    st = hntl.hntl_index_export(ix)
    grain = np.empty(ix.N, np.int32)
    grain[st["perm"]] = np.searchsorted(st["offsets"], np.arange(ix.N), side="right") - 1
    tg = to_dev(grain[ids.cpu().numpy()].astype(np.int32))
    kw = dict(hidden=(16, 8), epochs=2, batch=32, knn=kt, lr=1e-2, seed=3,
              flags=0 if shuffled else hntl.HNTL_ROUTER_NO_SHUFFLE)
    a = hntl.hntl_router_train(ix, X, targets=None, **kw)
    wa = hntl.hntl_router_export(ix)
    b = hntl.hntl_router_train(ix, X, targets=tg, **kw)
    wb = hntl.hntl_router_export(ix)
    for k in wa:
        np.testing.assert_array_equal(wa[k], wb[k])
    np.testing.assert_allclose(a, b, rtol=1e-5)  # a batch's losses are added in any order
