"""The ways out of the interior-point solve other than convergence, on chip and on
the elimination tree: a failed line search reports the KKT error of the point it
returns (that of the same solve stopped by its iteration limit there), a state
Jacobian that is singular or nearly so ends in a failed inertia correction or a
device error, and the handle's next solve is a new handle's.  And a solve on the
tree that corrects the inertia on its way to the solution."""
import dataclasses

import numpy as np
import pytest

import synthgrid as sg
from oracle import kkt, ipm
from test_gpu_solve_paths import _solve

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

TREE = dict(variant=1, col_tile=64, sweep_form=2)


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


def _create(inst, opts):
    import paper_2301_04869_amd as R
    return R, R.rkkt_create(inst.net, inst.scen.pd.T, inst.scen.qd.T, **opts)


@pytest.mark.parametrize("opts", [{}, TREE], ids=["chip", "tree"])
@pytest.mark.parametrize("name,n_scen", [("tiny9", 1), ("c0", 2)])
def test_line_search_failure_reports_its_point(name, n_scen, opts):
    """Line limits at a twentieth: no feasible point."""
    base = sg.preset(name, n_scen=n_scen)
    inst = dataclasses.replace(base, net=dataclasses.replace(base.net, rate=0.05 * base.net.rate))
    R, p = _create(inst, opts)
    res, out = _solve(p)
    assert res["status"] == "line_search_failed" and res["iters"] > 0
    lim, at = _solve(p, max_iter=res["iters"])
    assert lim["status"] == "max_iter"
    print(f"\n  {res['iters']} iterations, kkt error {res['kkt_error']:.6e}, stopped there {lim['kkt_error']:.6e}")
    assert res["kkt_error"] == lim["kkt_error"] and res["obj"] == lim["obj"]
    for k in out:
        assert torch.equal(out[k], at[k]), k
    if name == "c0":   # three iterations: the oracle takes the same ones
        ref = ipm.solve(kkt.Problem(inst))
        assert ref.status == "line_search_failed" and ref.iters == res["iters"]
        assert abs(res["kkt_error"] - ref.kkt_error) <= 1e-6 * ref.kkt_error


def _island(net, n):
    """n connected buses without a generator, and the lines between them."""
    pq = sorted(set(range(net.n_bus)) - set(map(int, net.gen_bus)))
    for a in pq:
        inside = [a] if n == 1 else next(([a, b] for b in pq if any(
            {int(f), int(t)} == {a, b} for f, t in zip(net.line_from, net.line_to))), None)
        if inside:
            ends = np.array([[int(f) in inside, int(t) in inside]
                             for f, t in zip(net.line_from, net.line_to)])
            return ends.any(axis=1) & ~ends.all(axis=1)
    raise AssertionError("no such buses")


@pytest.mark.parametrize("opts", [{}, TREE], ids=["chip", "tree"])
@pytest.mark.parametrize("n,left,status", [(1, 0.0, "inertia_correction_failed"), (2, 1e-13, "device_error")])
def test_singular_state_jacobian_ends_the_solve(n, left, status, opts):
    """Buses whose lines to the rest of the grid are out of service (the pivots
    are zero and K_hat is not a number), or nearly so (a pivot fails the health
    test and K_hat still factorises)."""
    inst = sg.preset("c0", n_scen=2)
    R, p = _create(inst, opts)
    st = torch.ones(2, inst.net.n_line, dtype=torch.float64, device="cuda")
    st[1, torch.tensor(_island(inst.net, n), device="cuda")] = left
    R.rkkt_set_line_status(p, st)
    res, _ = _solve(p)
    print(f"\n  {res}")
    assert res["status"] == status and res["iters"] == 0
    # the raised status stays for the caller unless the solve reported it
    assert R.rkkt_status(p)[0] == (-3 if status == "inertia_correction_failed" else 0)
    R.rkkt_set_line_status(p, torch.ones_like(st))
    _, q = _create(inst, opts)
    (ra, a), (rb, b) = _solve(p), _solve(q)
    assert ra == rb and ra["status"] == "converged"
    for k in a:
        assert torch.equal(a[k], b[k]), k


def test_inertia_correction_on_the_tree():
    inst = sg.preset("c0")
    ref = ipm.solve(kkt.Problem(inst))
    R, p = _create(inst, TREE)
    res, out = _solve(p)
    print(f"\n  {res}")
    assert ref.status == res["status"] == "converged"
    assert res["factorizations"] > res["iters"]
    # as in test_gpu_ipm
    assert abs(res["iters"] - ref.iters) <= 2
    assert abs(res["obj"] - ref.obj) <= 1e-6 * abs(ref.obj)
    assert np.abs(out["u"].cpu().numpy() - ref.it.u).max() <= 1e-5
