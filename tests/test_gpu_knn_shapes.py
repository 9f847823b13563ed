"""GPU tests of neighbour searches at the sizes where the tile form and the number
of column ranges change, on whole numbers whose distances are exact, and of the
time of a small search against that of its smallest form."""
import numpy as np
import pytest

from tests.gpu_common import announce, require_gpu
from tests.test_gpu_knn_ties import flat_index

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nq,N,d", [
    (16, 1537, 40), (17, 1537, 40), (90, 1500, 768), (448, 2304, 384), (447, 2304, 384), (448, 25_601, 384),
    (700, 9000, 640), (449, 2240, 400), (1500, 700, 256), (3000, 1153, 64), (1, 33_000, 32), (65, 65_000, 32),
    (300, 45_000, 256), (2049, 12_800, 160), (1024, 6000, 512), (130, 1920, 36)])
def test_every_form_and_range_count(nq, N, d):
    torch = require_gpu()
    from paper_2606_08813_amd import hntl
    announce(f"neighbours of {nq} rows among {N} x {d}")
    g = torch.Generator(device="cuda").manual_seed(N + nq)
    X = torch.randint(-6, 7, (N, d), device="cuda", generator=g).float()
    Q = torch.randint(-6, 7, (nq, d), device="cuda", generator=g).float()
    ids, dist = hntl.hntl_knn(flat_index(hntl, torch, X), Q, 10)
    Xd, x2 = X.double(), (X.double() ** 2).sum(1)
    for a in range(0, nq, 256):
        q = Q[a:a + 256].double()
        D = (q ** 2).sum(1, keepdim=True) + x2 - 2.0 * (q @ Xd.t())  # whole numbers below 2^53: exact
        order = (D * 2.0 ** 20 + torch.arange(N, device="cuda", dtype=torch.float64)).topk(10, largest=False, sorted=True)
        assert torch.equal(ids[a:a + 256].long(), order.indices)
        assert torch.equal(dist[a:a + 256].double(), D.gather(1, order.indices))


def test_a_small_search_is_spread_over_the_gpu():
    torch = require_gpu()
    from paper_2606_08813_amd import hntl
    announce("1 and 128 queries over 2,000 x 768 rows")
    g = torch.Generator(device="cuda").manual_seed(3)
    ix = flat_index(hntl, torch, torch.randn(2000, 768, device="cuda", generator=g))

    def best(nq):
        Q = torch.randn(nq, 768, device="cuda", generator=g)
        t = []
        for _ in range(15):
            a, b = torch.cuda.Event(True), torch.cuda.Event(True)
            a.record()
            hntl.hntl_knn(ix, Q, 10)
            b.record()
            torch.cuda.synchronize()
            t.append(a.elapsed_time(b))
        return min(t[3:])
    one, many = best(1), best(128)
    # 1.1 of it; 3.0 where a workgroup took 64 rows and eight tiles of columns at least
    assert many < 1.8 * one, (many, one)
