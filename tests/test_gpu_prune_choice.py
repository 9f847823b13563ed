"""GPU tests of when a plan prunes pairs before their projection: where grains lie
apart the other slots' pairs are dropped unscanned, where they overlap the plan
takes no second bucketing, projection and scan for what it would keep anyway."""
import numpy as np
import pytest

from tests.gpu_common import announce, require_gpu

pytestmark = pytest.mark.gpu

P, C, K = 8, 20, 10


def apart(torch, hntl, N, G, d, r):
    """Far apart grains of equal size, codes of a few units."""
    g = torch.Generator(device="cuda").manual_seed(1)
    cent = 4.0 * torch.randn(G, d, device="cuda", generator=g)
    W = torch.zeros(G, r, d, device="cuda")
    W[:, torch.arange(r), torch.arange(r)] = 1.0
    z = torch.randn(N, r, device="cuda", generator=g)
    lab = torch.arange(N, device="cuda") * G // N
    X = cent[lab]
    X[:, :r] += z
    off = np.searchsorted(lab.cpu().numpy(), np.arange(G + 1)).astype(np.int64)
    st = dict(centroids=cent, basis=W, offsets=off, perm=np.arange(N, dtype=np.int32), codes=z.cpu().numpy(),
              eps=np.zeros(N, np.float32))
    return hntl.hntl_index_create(st, X), X, off


@pytest.mark.parametrize("nq,prunes", [(1500, False), (2000, True)])  # 10,500 and 14,000 pairs
def test_grains_apart(nq, prunes):
    torch = require_gpu()
    from paper_2606_08813_amd import hntl
    announce(f"plan of {nq} over grains apart")
    ix, X, off = apart(torch, hntl, 40_000, 100, 32, 16)
    Q = X[:: len(X) // nq][:nq].contiguous()
    for sched in (dict(qt=2, nw=2, range=0, passes=1, proj=1), dict(qt=2, nw=2, range=0, passes=1, proj=0)):
        plan = hntl.hntl_plan_create(ix, P, C, K, nq, sched=sched)
        got = hntl.hntl_plan_search(plan, Q)
        want = hntl.hntl_search(ix, Q, P, C, K, flags=hntl.HNTL_FLAG_SYNC | hntl.HNTL_FLAG_NO_PRUNE)
        assert torch.equal(got[0], want[0]) and torch.equal(got[1], want[1])
        _, scored = hntl.hntl_plan_profile(plan, nq, reps=1)
        own = np.searchsorted(off, np.arange(0, len(X), len(X) // nq)[:nq], side="right") - 1
        first = int((off[own + 1] - off[own]).sum())
        # with every item in one launch the first waves find no bound yet
        assert (scored == first) == (prunes and sched["proj"] == 1), (scored, first, sched)


def test_overlapping_grains_cost_no_second_pass():
    torch = require_gpu()
    from paper_2606_08813_amd import hntl
    announce("plan of 100 over 1,024 grains of one cloud")
    d = 768
    g = torch.Generator(device="cuda").manual_seed(2)
    scale = torch.arange(1, d + 1, device="cuda", dtype=torch.float32) ** -0.5
    X = (torch.randn(60_000, d, device="cuda", generator=g) * scale).contiguous()
    Q = (torch.randn(100, d, device="cuda", generator=g) * scale).contiguous()
    ix = hntl.hntl_build(X, 1024, 48, kmeans_iters=3, eig_iters=4)

    def best(flags):
        plan = hntl.hntl_plan_create(ix, P, C, K, len(Q), flags=flags)
        t = []
        for _ in range(30):
            a, b = torch.cuda.Event(True), torch.cuda.Event(True)
            a.record()
            r = hntl.hntl_plan_search(plan, Q)
            b.record()
            torch.cuda.synchronize()
            t.append(a.elapsed_time(b))
        return min(t), r
    with_prune, a = best(0)
    without, b = best(hntl.HNTL_FLAG_NO_PRUNE)
    assert torch.equal(a[0], b[0]) and torch.equal(a[1], b[1])
    assert with_prune < 1.15 * without, (with_prune, without)  # 1.3 with both passes


def test_tuner_times_a_pipeline_once():
    torch = require_gpu()
    from paper_2606_08813_amd import hntl
    announce("tuning where plans prune pairs and passes is not read")
    ix, X, _ = apart(torch, hntl, 20_000, 50, 32, 16)
    for nq in (2000, 2100, 2200, 2300, 2400):
        best, ms = hntl.hntl_tune(ix, X[:nq].contiguous(), P, C, K)
        assert ms > 0 and not (best["proj"] == 1 and best["passes"] == 2), best
