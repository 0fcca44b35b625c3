"""The blocked Cholesky where a pivot fails: what the launches before the failing
tile have finished does not depend on when a workgroup sees the failure.  With
the first bad pivot in 64-column tile t, the panels before t - 1 hold the factor
of the leading columns (all rows), and repeated factorisations leave the same
bits everywhere."""
import numpy as np
import pytest
import scipy.linalg as sla

import gpu_common as gc
from test_gpu_chol import _handle

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


@pytest.mark.parametrize("n,col", [(129, 100), (257, 130), (641, 450), (1281, 640), (1281, 1281)])
def test_failed_factor_is_deterministic(n, col):
    R, p = _handle(n)
    rng = np.random.default_rng(n + col)
    m = rng.standard_normal((n, n))
    a = m @ m.T / n + np.eye(n)
    ref_a = a.copy()
    a[col - 1, col - 1] = -1.0
    src = torch.tensor(a, device="cuda")
    info = torch.zeros(1, dtype=torch.int32, device="cuda")
    got = []
    for _ in range(20):
        dev = src.clone()
        R.rkkt_factor(p, dev, info)
        assert int(info.item()) == col
        got.append(dev)
    assert all(torch.equal(got[0], g) for g in got[1:])
    t = (col - 1) // 64
    lead = 64 * max(0, t - 1)
    if lead:
        # the rows and columns before the bad pivot are those of a definite
        # matrix: its factor's leading columns, within a block factorisation's
        # backward error times the conditioning
        k = col - 1
        ref = sla.cholesky(ref_a[:k, :k], lower=True)[:, :lead]
        L = np.tril(got[0].cpu().numpy())[:k, :lead]
        assert gc.rel_fro(L, ref) <= 4 * k * gc.EPS * gc.cond2(ref_a[:k, :k])
