"""GPU tests of the projection at the row lengths and ranks where its depth
chunks, its prefetch rule and its 16-row basis tiles end, against float64."""
import numpy as np
import pytest

from tests.gpu_common import announce, require_gpu, to_dev
from workloads import patch_mixture as pm

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d,r", [(16, 8), (60, 16), (68, 17), (128, 32), (252, 24), (256, 16), (260, 32), (264, 33),
                                 (320, 48), (324, 32), (764, 30), (768, 64)])
@pytest.mark.parametrize("bf16", [False, True], ids=["fp32", "bf16"])
def test_tangents(d, r, bf16):
    torch = require_gpu()
    from paper_2606_08813_amd import hntl
    if bf16 and d % 8:
        pytest.skip("BF16 projection takes d % 8 == 0")
    announce(f"projection of d = {d} at rank {r}, bf16 {bf16}")
    G, nq, P, N = 9, 130, 4, 900
    rng = np.random.default_rng(101)
    W = np.stack([np.linalg.qr(rng.standard_normal((d, r)))[0].T for _ in range(G)]).astype(np.float32)
    cent = pm.uniform_rows(G, d, 102)
    X = pm.uniform_rows(N, d, 103)
    st = dict(centroids=cent, basis=W, offsets=(np.arange(G + 1, dtype=np.int64) * N) // G,
              perm=np.arange(N, dtype=np.int32), codes=pm.uniform_floats((N, r), 104), eps=np.ones(N, np.float32))
    ix = hntl.hntl_index_create(st, X, codes=("fp32", "bf16") if bf16 else ("fp32",))
    Q = pm.uniform_rows(nq, d, 105)
    o = hntl.hntl_search_stages(ix, to_dev(Q), P, 8, 1,
                                flags=hntl.HNTL_FLAG_SYNC | (hntl.HNTL_FLAG_PROJECT_BF16 if bf16 else 0))
    pr, z, e = (o[k].cpu().numpy() for k in ("probes", "zq", "epsq"))
    qc = Q[:, None, :] - cent[pr]  # FP32, as formed on the device
    Wr = W[pr]
    if bf16:
        rnd = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to(torch.bfloat16).float().numpy()
        qr, Wr = rnd(qc), rnd(Wr)
    else:
        qr = qc
    ref = np.einsum("qpd,qprd->qpr", qr.astype(np.float64), Wr.astype(np.float64))
    nrm = np.linalg.norm(qc.astype(np.float64), axis=2)
    # sums of d FP32 products of rows of norm 1 and |q'|: d 2^-24 |q'|
    assert (np.abs(z - ref) <= d * 2.0 ** -24 * nrm[..., None]).all()
    eref = np.maximum(nrm ** 2 - (z.astype(np.float64) ** 2).sum(2), 0.0)
    assert (np.abs(e - eref) <= 2 * d * 2.0 ** -24 * nrm ** 2).all()
