"""The interior-point solve where its paths differ: scenario counts whose
reductions take one workgroup and several, the reduction's variants (the
elimination tree included), an iteration limit that ends the solve with a
refactorisation in flight, and the handle's state afterwards.  Against the
oracle's outer loop as in test_gpu_ipm (iterations within 2, objective 1e-6
relative, controls 1e-5); a second solve on the same handle is equal bit for
bit, and the device status is clear after a solve."""
import numpy as np
import pytest

import synthgrid as sg
from oracle import kkt, ipm

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


def _solve(p, **k):
    d = p.dims
    n = d["n_scen"]
    out = {a: torch.zeros(s, dtype=torch.float64, device="cuda")
           for a, s in dict(x=(n, d["n_x"]), u=d["n_u"], y=(n, d["n_x"]), z=(n, d["m"]), s=(n, d["m"])).items()}
    return __import__("paper_2301_04869_amd").rkkt_solve(p, **out, **k), out


@pytest.mark.parametrize("name,n_scen,opts", [
    ("tiny9", 1, {}),
    ("c0", 40, {}),                                          # merit over several workgroups
    ("c0", 3, dict(variant=1)),
    ("c0", 3, dict(variant=1, col_tile=64, sweep_form=2)),   # elimination tree
])
def test_solve_paths(name, n_scen, opts):
    import paper_2301_04869_amd as R
    inst = sg.preset(name, n_scen=n_scen)
    ref = ipm.solve(kkt.Problem(inst))
    assert ref.status == "converged"
    p = R.rkkt_create(inst.net, inst.scen.pd.T, inst.scen.qd.T, **opts)
    res, out = _solve(p)
    assert res["status"] == "converged"
    assert res["kkt_error"] <= 1e-8
    assert abs(res["iters"] - ref.iters) <= 2
    assert abs(res["obj"] - ref.obj) <= 1e-6 * abs(ref.obj)
    assert np.abs(out["u"].cpu().numpy() - ref.it.u).max() <= 1e-5
    assert R.rkkt_status(p)[0] == 0
    res2, out2 = _solve(p)
    assert res2 == res
    for k in out:
        assert torch.equal(out[k], out2[k]), k


@pytest.mark.parametrize("limit", [0, 3])
def test_iteration_limit(limit):
    import paper_2301_04869_amd as R
    inst = sg.preset("c0")
    p = R.rkkt_create(inst.net, inst.scen.pd.T, inst.scen.qd.T)
    res, out = _solve(p, max_iter=limit)
    assert res["status"] == "max_iter" and res["iters"] == limit
    assert np.isfinite(res["kkt_error"]) and res["kkt_error"] > 1e-8
    assert R.rkkt_status(p)[0] == 0
    # the handle's next solve is that of a new handle
    q = R.rkkt_create(inst.net, inst.scen.pd.T, inst.scen.qd.T)
    (ra, a), (rb, b) = _solve(p), _solve(q)
    assert ra == rb and ra["status"] == "converged"
    for k in a:
        assert torch.equal(a[k], b[k]), k
