"""The blocked Cholesky and the reduced solve beyond 128 columns on ill-conditioned
matrices.  Both apply explicit inverses of diagonal blocks (16 x 16 in the factor,
64 x 64 in the solve) where substitution would divide, so what is checked is the
backward error, which conditioning must not enter: of the factor relative to |A|
and, scaled by the diagonal, entry by entry, and of the solve relative to
|A| |x| in norm and row by row."""
import numpy as np
import pytest

import gpu_common as gc
from test_gpu_chol import _handle

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


def _matrix(n, cond, kind, rng):
    """Eigenvalues spread evenly over the decades, five small ones, or a well
    conditioned matrix whose rows and columns are scaled over the decades."""
    q, _ = np.linalg.qr(rng.standard_normal((n, n)))
    lam = {"spread": np.logspace(0, -np.log10(cond), n), "few": np.where(np.arange(n) < n - 5, 1.0, 1.0 / cond),
           "graded": np.linspace(1.0, 2.0, n)}[kind]
    a = (q * lam) @ q.T
    if kind == "graded":
        s = np.logspace(0, -0.5 * np.log10(cond), n)[rng.permutation(n)]
        a = a * s[:, None] * s
    return (a + a.T) / 2


@pytest.mark.parametrize("kind", ["spread", "few", "graded"])
@pytest.mark.parametrize("cond", [1e8, 1e12])
@pytest.mark.parametrize("n", [129, 257, 641])
def test_backward_errors(n, cond, kind):
    R, p = _handle(n)
    d = p.dims
    nx, m = d["n_x"], d["m"]
    rng = np.random.default_rng([n, int(np.log10(cond)), len(kind)])
    a, b = _matrix(n, cond, kind, rng), rng.standard_normal(n)
    z = lambda *s: torch.zeros(*s, dtype=torch.float64, device="cuda")  # noqa: E731
    # a regular state: the step's other right-hand sides are zero
    x0, u0, one = z(1, nx), z(n), z(1, m) + 1.0
    x0[:, d["n_bus"] - 1:] = 1.0
    u0[:d["n_gen"]] = 1.0
    R.rkkt_evaluate(p, x0, u0, z(1, nx), z(1, m), 1.0, z(1), z(1, nx), z(1, n), z(1, nx), z(1, m))
    R.rkkt_condense(p, z(1, nx) + 1.0, z(n) + 1.0, one, 1.0, z(n, n))
    chol, info, pu = torch.tensor(a, device="cuda"), torch.zeros(1, dtype=torch.int32, device="cuda"), z(n)
    R.rkkt_factor(p, chol, info)
    R.rkkt_step(p, z(1, nx), torch.tensor(-b, device="cuda"), z(1, m), z(1, nx), z(1, m), one, chol, z(1, nx), pu,
                z(1, m), z(1, nx), z(1, m))
    torch.cuda.synchronize()
    assert int(info.item()) == 0
    L, x = np.tril(chol.cpu().numpy()), pu.cpu().numpy()
    dg = np.sqrt(np.diag(a))
    e = L @ L.T - a
    r = b - a @ x
    err = dict(factor=np.linalg.norm(e) / np.linalg.norm(a), scaled=np.abs(e / dg[:, None] / dg).max(),
               solve=np.linalg.norm(r) / (np.linalg.norm(a, 2) * np.linalg.norm(x) + np.linalg.norm(b)),
               rows=(np.abs(r) / (np.abs(a) @ np.abs(x) + np.abs(b))).max())
    print(f"\n  n {n} {kind} {cond:.0e}: " + " ".join(f"{k} {v:.1e}" for k, v in err.items()))
    # as in test_gpu_chol: a few n eps
    assert all(v <= 4 * n * gc.EPS for v in err.values()), err
