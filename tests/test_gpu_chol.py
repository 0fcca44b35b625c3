"""The blocked Cholesky and the reduced solve beyond 128 columns, alone: factor
of a seeded positive definite matrix against LAPACK, in place, the first
non-positive pivot reported from any panel, and the solve through rkkt_step
against the oracle is covered by the step tests; here the orders at the edges
of the 64-column tiles and of the solve's panels (10 tiles)."""
import numpy as np
import pytest
import scipy.linalg as sla

import gpu_common as gc
import synthgrid as sg

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


def _handle(n_u, n_scen=1):
    """A handle with n_u = 2 n_gen - 1 controls (a path of generator buses)."""
    import paper_2301_04869_amd as R
    ng = (n_u + 1) // 2
    net = sg.make_network(ng + 2, ng + 1, ng, 5)
    scen = sg.make_scenarios(net, n_scen, 0.1, 6)
    return R, R.rkkt_create(net, scen.pd.T, scen.qd.T)


@pytest.mark.parametrize("n", [129, 191, 193, 255, 257, 319, 641, 1281])
def test_factor_matches_lapack(n):
    R, p = _handle(n)
    rng = np.random.default_rng(n)
    m = rng.standard_normal((n, n))
    a = m @ m.T / n + np.diag(rng.uniform(0.5, 2.0, n))
    dev = torch.tensor(a, device="cuda")
    info = torch.full((1,), -7, dtype=torch.int32, device="cuda")
    R.rkkt_factor(p, dev, info)
    torch.cuda.synchronize()
    assert int(info.item()) == 0
    L = np.tril(dev.cpu().numpy())
    # backward error of a factorisation by blocks: a few n eps |A|
    err = np.linalg.norm(L @ L.T - a) / np.linalg.norm(a)
    ref = sla.cholesky(a, lower=True)
    print(f"\n  n {n}: backward {err:.1e}, against LAPACK {gc.rel_fro(L, ref):.1e}")
    assert err <= 4 * n * gc.EPS
    assert gc.rel_fro(L, ref) <= 4 * n * gc.EPS * gc.cond2(a)
    # the strict upper triangle is the caller's
    assert np.array_equal(np.triu(dev.cpu().numpy(), 1), np.triu(a, 1))


@pytest.mark.parametrize("n,col", [(129, 1), (129, 65), (129, 129), (257, 64), (257, 200), (641, 577)])
def test_first_bad_pivot_is_reported(n, col):
    R, p = _handle(n)
    rng = np.random.default_rng(col)
    m = rng.standard_normal((n, n))
    a = m @ m.T / n + np.eye(n)
    a[col - 1, col - 1] = -1.0
    dev = torch.tensor(a, device="cuda")
    info = torch.zeros(1, dtype=torch.int32, device="cuda")
    R.rkkt_factor(p, dev, info)
    torch.cuda.synchronize()
    assert int(info.item()) == col


@pytest.mark.parametrize("n,n_scen", [(129, 1), (191, 3), (257, 9), (641, 2), (1281, 1)])
def test_step_solves_with_the_factor(n, n_scen):
    """p_u of rkkt_step with a given factor: the step is affine in r1u with
    slope -(L L^T)^-1, so two right-hand sides that differ in r1u alone give
    the solve by itself."""
    R, p = _handle(n, n_scen)
    d = p.dims
    nx, m = d["n_x"], d["m"]
    rng = np.random.default_rng(n + 1)
    q = rng.standard_normal((n, n))
    a = q @ q.T / n + np.diag(rng.uniform(0.5, 2.0, n))
    z = lambda *s: torch.zeros(*s, dtype=torch.float64, device="cuda")  # noqa: E731
    net_x = z(n_scen, nx)
    net_x[:, :] = 1.0
    net_x[:, :d["n_bus"] - 1] = 0.0
    u = z(n)
    u[:d["n_gen"]] = 1.0
    R.rkkt_evaluate(p, net_x, u, z(n_scen, nx), z(n_scen, m), 1.0, z(n_scen), z(n_scen, nx), z(n_scen, n),
                    z(n_scen, nx), z(n_scen, m))
    one = torch.ones(n_scen, m, dtype=torch.float64, device="cuda")
    R.rkkt_condense(p, z(n_scen, nx) + 1.0, z(n) + 1.0, one, 1.0, z(n, n))
    chol = torch.tensor(a, device="cuda")
    info = torch.zeros(1, dtype=torch.int32, device="cuda")
    R.rkkt_factor(p, chol, info)
    b = rng.standard_normal(n)
    out = []
    for r1u in (np.zeros(n), b):
        pu = z(n)
        R.rkkt_step(p, z(n_scen, nx), torch.tensor(r1u, device="cuda"), z(n_scen, m), z(n_scen, nx), z(n_scen, m),
                    one, chol, z(n_scen, nx), pu, z(n_scen, m), z(n_scen, nx), z(n_scen, m))
        out.append(pu.cpu().numpy())
    got, ref = out[1] - out[0], -sla.cho_solve((sla.cholesky(a, lower=True), True), b)
    err = np.linalg.norm(got - ref) / np.linalg.norm(ref)
    print(f"\n  n {n} N {n_scen}: {err:.1e}")
    assert err <= 4 * n * gc.EPS * gc.cond2(a)
