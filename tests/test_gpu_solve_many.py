"""The interior-point step where the step lengths come from more than 2048 partial
reductions (k_step_fin): the first iteration over 900 scenarios of the 118-bus grid
against the same iteration put together from the library's four calls and the
oracle's start point, residuals and step-length rule, all scenarios at once."""
import numpy as np
import pytest

import synthgrid as sg
from oracle import kkt, ipm
from test_gpu_solve_paths import _solve

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


def test_step_lengths_of_many_scenarios():
    import paper_2301_04869_amd as R
    n = 900
    inst = sg.preset("c1", n_scen=n)
    p = R.rkkt_create(inst.net, inst.scen.pd.T, inst.scen.qd.T)
    d, opt = p.dims, ipm.Options()
    nx, nu, m = d["n_x"], d["n_u"], d["m"]
    assert n * (nx + m) + nu > 2048 * 256
    prob = kkt.Problem(inst)
    one, _ = ipm.initial_point(kkt.Problem(sg.preset("c1", n_scen=1)), opt)
    # the start point of the cold solve
    dev = lambda a: torch.tensor(a, dtype=torch.float64, device="cuda")  # noqa: E731
    z = lambda *s: torch.zeros(*s, dtype=torch.float64, device="cuda")  # noqa: E731
    x0, u0 = np.tile(one.x, (n, 1)), one.u
    f, gx, gu, g, h = z(n), z(n, nx), z(n, nu), z(n, nx), z(n, m)

    def evaluate(w):
        R.rkkt_evaluate(p, dev(x0), dev(u0), z(n, nx), z(n, m), w, f, gx, gu, g, h)
        torch.cuda.synchronize()
    evaluate(1.0 / n)
    gmax = max(float(gx.abs().max()), float(gu.sum(0).abs().max()))
    w = min(1.0, opt.obj_scale_max_grad / gmax) / n
    s0 = ipm._push(-h.cpu().numpy(), prob.sl, prob.su, opt.kappa1, opt.kappa2)
    evaluate(w)
    on = lambda b: np.isfinite(b) * 1.0  # noqa: E731  (bound multipliers 1)
    parts = {k: kkt._bound_parts(v, lo, hi, on(lo), on(hi), opt.mu0)
             for k, v, lo, hi in (("x", x0, prob.xl, prob.xu), ("u", u0, prob.ul, prob.uu),
                                  ("s", s0, prob.sl, prob.su))}
    (sx, bx), (su, bu), (ss, bs) = parts["x"], parts["u"], parts["s"]
    khat, info = z(nu, nu), torch.zeros(1, dtype=torch.int32, device="cuda")
    R.rkkt_condense(p, dev(sx), dev(su), dev(ss), 0.0, khat)
    R.rkkt_factor(p, khat, info)
    px, pu, ps, py, pz = z(n, nx), z(nu), z(n, m), z(n, nx), z(n, m)
    R.rkkt_step(p, gx + dev(bx), gu.sum(0) + dev(bu), dev(bs), g, h + dev(s0), dev(ss), khat, px, pu, ps, py, pz)
    torch.cuda.synchronize()
    assert int(info.item()) == 0 and R.rkkt_status(p)[0] == 0
    tau = max(opt.tau_min, 1.0 - opt.mu0)
    step = {"x": px.cpu().numpy(), "u": pu.cpu().numpy(), "s": ps.cpu().numpy()}
    a = min(ipm._max_step(x0, step["x"], prob.xl, prob.xu, tau), ipm._max_step(u0, step["u"], prob.ul, prob.uu, tau),
            ipm._max_step(s0, step["s"], prob.sl, prob.su, tau))
    res, out = _solve(p, max_iter=1)
    assert res["status"] == "max_iter" and res["iters"] == 1 and res["factorizations"] == 1
    # the accepted step is the largest one, or that halved by the line search
    du = out["u"].cpu().numpy() - u0
    halvings = round(np.log2(a * np.linalg.norm(step["u"]) / np.linalg.norm(du)))
    a *= 0.5 ** halvings
    print(f"\n  step length {a:.6f} after {halvings} halvings")
    assert 0 <= halvings <= 3
    # two FP64 computations of one Newton step
    bar = max(1e-10, 10 * np.finfo(float).eps * np.linalg.cond(np.tril(khat.cpu().numpy())) ** 2)
    for k, v, at in (("x", x0, out["x"]), ("u", u0, out["u"]), ("s", s0, out["s"])):
        err = np.linalg.norm(at.cpu().numpy() - v - a * step[k]) / np.linalg.norm(a * step[k])
        print(f"  {k}: {err:.1e} (bar {bar:.1e})")
        assert err <= bar
    again, out2 = _solve(p, max_iter=1)
    assert again == res and all(torch.equal(out[k], out2[k]) for k in out)
