"""The work that users of this library have it do, as cases that can be timed.

A case is one pass through the public entry points on inputs made from a seed:

* ``pass``: one interior-point iteration's linear algebra of a block AC-OPF
  (evaluate, condense, factor, step) over N load scenarios of one grid, as a
  captured graph, as one eager call, or as the four separate calls;
* ``multi``: the same pass for several independent grids of uneven sizes;
* ``solve``: a whole interior-point solve;
* ``forward`` / ``train``: the warm-start perceptron's forward pass, and its
  loss, gradients and Adam step.

Grids are drawn by the benchmark's recipe (random geometric tree and chords,
its parameter distributions) with the bus / line / generator counts of its
workloads.  ``exact`` computes the same outputs densely in 64 bits.
"""
from __future__ import annotations

import functools
import math
from types import SimpleNamespace

import numpy as np
import torch

import paper_2301_04869_amd as R

F64 = torch.float64


def listed():
    return [
        # the smallest call: a 30-bus grid, one scenario, replayed as a graph;
        # launches and latency are all there is
        dict(name="pass 30 bus x 1 graph", kind="pass", buses=30, lines=41, gens=6, loads=24, scen=1,
             delta_w=0.0, how="graph"),
        # the four calls one after the other, as a caller's own solver loop
        # makes them on one load draw of the 118-bus grid
        dict(name="pass 118 bus x 1 calls", kind="pass", buses=118, lines=186, gens=54, loads=99, scen=1,
             delta_w=1.0, how="calls"),
        # the benchmark's default workload
        dict(name="pass 118 bus x 128 graph", kind="pass", buses=118, lines=186, gens=54, loads=99, scen=128,
             delta_w=0.0, how="graph"),
        # the largest scenario counts that the 118-bus grid is used with, an
        # odd count, as one eager call
        dict(name="pass 118 bus x 1001 eager", kind="pass", buses=118, lines=186, gens=54, loads=99, scen=1001,
             delta_w=1.0, how="eager"),
        # a middle-sized grid (the tests' 300-bus grid) with a few scenarios
        dict(name="pass 300 bus x 16 graph", kind="pass", buses=300, lines=450, gens=80, loads=220, scen=16,
             delta_w=1.0, how="graph"),
        # 8 scenarios of the 1354-, 2869- and 16 of the 9241-bus grids of the
        # paper's tables
        dict(name="pass 1354 bus x 8 graph", kind="pass", buses=1354, lines=1991, gens=260, loads=1094, scen=8,
             delta_w=1.0, how="graph"),
        dict(name="pass 2869 bus x 8 eager", kind="pass", buses=2869, lines=4582, gens=510, loads=2359, scen=8,
             delta_w=1.0, how="eager"),
        dict(name="pass 9241 bus x 16 graph", kind="pass", buses=9241, lines=16049, gens=1445, loads=7796,
             scen=16, delta_w=1.0, how="graph"),
        # independent single-scenario grids of 300 to 2000 buses in one launch
        # set (the generation of warm-start data)
        dict(name="multi 16 grids", kind="multi", count=16, low=300, high=2000, delta_w=1.0, how="graph"),
        # one cold solve of a load draw: what generating warm-start data repeats
        dict(name="solve 118 bus x 1", kind="solve", buses=118, lines=186, gens=54, loads=99, scen=1,
             sigma=0.1),
        # the perceptron: a prediction for 256 load draws, one training step
        dict(name="forward 256", kind="forward", batch=256, inputs=198, hidden=512, outputs=896),
        dict(name="train 256", kind="train", batch=256, inputs=198, hidden=512, outputs=896),
    ]


def draw(rng):
    """Another case of the listed ranges; sizes over their logarithm."""
    def size(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))
    kind = rng.choice(("pass", "pass", "pass", "pass", "multi", "solve", "forward", "train"))
    if kind == "pass":
        nb = size(30, 4000)
        # scenario counts up to 1001, and no more than the work of the largest case
        ns = size(1, min(1001, max(2.0, 1.2e5 / nb)))
        ng = max(3, int(nb * rng.uniform(0.12, 0.4 if nb < 400 else 0.2)))
        return dict(kind=kind, buses=nb, lines=int(nb * rng.uniform(1.35, 1.75)), gens=ng,
                    loads=int((nb - ng) * rng.uniform(0.8, 1.0)), scen=ns, delta_w=1.0,
                    how=rng.choice(("graph", "graph", "eager", "calls")))
    if kind == "multi":
        return dict(kind=kind, count=size(2, 16), low=size(100, 400), high=size(600, 2000), delta_w=1.0,
                    how=rng.choice(("graph", "eager")))
    if kind == "solve":
        # the grid whose solves converge from the flat start, wider or narrower load draws
        return dict(kind=kind, buses=118, lines=186, gens=54, loads=99, scen=1, sigma=rng.uniform(0.04, 0.15))
    return dict(kind=kind, batch=size(1, 512), inputs=2 * size(20, 99), hidden=32 * rng.randint(4, 16),
                outputs=rng.randint(200, 896))


# ------------------------------------------------------------------ the inputs
@functools.lru_cache(maxsize=40)
def _grid(nb, nl, ng, nload, seed=0):
    """One grid of the benchmark's recipe: buses uniform in the unit square,
    each new bus tied to one of its 3 nearest earlier ones, chords among the 6
    nearest neighbours, generators at spread-out buses."""
    rng = np.random.default_rng([seed, nb, nl, ng])
    xy = rng.random((nb, 2))
    edges, near = set(), []
    for t in range(nb):
        d2 = ((xy - xy[t]) ** 2).sum(axis=1)
        d2[t] = np.inf
        if t:
            c = np.argsort(d2[:t])[:3] if t < 40 else np.argpartition(d2[:t], 2)[:3]
            edges.add((int(c[rng.integers(len(c))]), t))
        near.append(np.argpartition(d2, min(6, nb - 1) - 1)[:6])
    while len(edges) < nl:
        a = int(rng.integers(nb))
        c = int(near[a][rng.integers(len(near[a]))])
        edges.add((min(a, c), max(a, c)))
    e = np.array(sorted(edges), dtype=np.int32)
    e = np.where((rng.random(nl) < 0.5)[:, None], e[:, ::-1], e)[rng.permutation(nl)]
    chosen = [int(rng.integers(nb))]
    dist = ((xy - xy[chosen[0]]) ** 2).sum(axis=1)
    while len(chosen) < ng:
        cand = rng.choice(nb, size=min(8, nb), replace=False)
        best = int(cand[np.argmax(dist[cand])])
        if dist[best] > 0:
            chosen.append(best)
            dist = np.minimum(dist, ((xy - xy[best]) ** 2).sum(axis=1))
    gen = np.sort(np.array(chosen, dtype=np.int32))
    free = np.setdiff1d(np.arange(nb), gen)
    load = np.sort(free[rng.permutation(len(free))[:nload]] if nload <= len(free)
                   else rng.choice(nb, size=nload, replace=False)).astype(np.int32)
    pd = rng.uniform(0.1, 0.5, nload) * (1.0 if nb <= 500 else 0.15)
    cell = np.bincount([int(np.argmin(((xy[gen] - xy[b]) ** 2).sum(axis=1))) for b in load], weights=pd,
                       minlength=ng)
    pmax = (cell + 0.25 * pd.sum() / ng) * rng.uniform(0.5, 1.5, ng)
    pmax *= 2.0 * pd.sum() / pmax.sum()
    gref = int(np.argmax(pmax))
    pmax[gref] += max(1.0, 0.6 * math.sqrt((pd ** 2).sum()))
    f, t = np.ascontiguousarray(e[:, 0]), np.ascontiguousarray(e[:, 1])
    x = rng.uniform(0.05, 0.4, nl)
    rate = np.full(nl, 3.0)
    if nb <= 500:  # limits that a DC flow at proportional dispatch keeps with a margin
        B = np.zeros((nb, nb))
        for a, b, w in ((f, t, -1.0), (t, f, -1.0), (f, f, 1.0), (t, t, 1.0)):
            np.add.at(B, (a, b), w / x)
        inj = np.zeros(nb)
        disp = pmax.copy()
        disp[gref] = np.median(pmax)
        inj[gen] += disp * (pd.sum() / disp.sum())
        np.add.at(inj, load, -pd)
        keep = np.arange(nb) != gen[gref]
        th = np.zeros(nb)
        th[keep] = np.linalg.solve(B[np.ix_(keep, keep)], inj[keep])
        rate = np.maximum(0.3, rng.uniform(1.5, 2.5, nl) * np.abs((th[f] - th[t]) / x) + 0.1)
    return SimpleNamespace(
        n_bus=nb, n_line=nl, n_gen=ng, ref_bus=int(gen[gref]), gref=gref, line_from=f, line_to=t,
        r=rng.uniform(0.01, 0.1, nl), x=x, b=rng.uniform(0.0, 0.05, nl), rate=rate, gen_bus=gen,
        pmin=np.zeros(ng), pmax=pmax, qmin=-0.5 * pmax, qmax=0.5 * pmax, c2=rng.uniform(0.01, 0.1, ng),
        c1=rng.uniform(10.0, 40.0, ng), c0=np.zeros(ng), vmin=np.full(nb, 0.9), vmax=np.full(nb, 1.1),
        load_bus=load, pd=pd, qd=0.3 * pd)


def _grids(c):
    """The grids of a case, each with its scenario count."""
    if c["kind"] == "multi":
        rng = np.random.default_rng([c["count"], c["low"], c["high"]])
        sizes = np.exp(rng.uniform(math.log(c["low"]), math.log(c["high"]), c["count"])).round().astype(int)
        return [(_grid(int(nb), round(1.5 * nb), round(0.15 * nb), int(nb) - round(0.15 * nb), j), 1)
                for j, nb in enumerate(sizes)]
    return [(_grid(c["buses"], c["lines"], c["gens"], c["loads"]), c["scen"])]


def _sizes(net):
    return 2 * net.n_bus - net.n_gen - 1, 2 * net.n_gen - 1, 2 * net.n_line + net.n_gen + 1


def _loads(net, ns, rng, sigma=0.1):
    """Load draws: the base loads times clip(1 + sigma xi, 0.5, 1.5)."""
    fac = np.clip(1.0 + sigma * rng.standard_normal((ns, len(net.load_bus))), 0.5, 1.5)
    return net.pd * fac, net.qd * fac


def _iterate(net, ns, rng):
    """An interior-point iterate's values: angles and magnitudes about the
    flat start, outputs inside their boxes, multipliers of an objective
    weighted 1/N, diagonals over two decades, Newton residuals."""
    nx, nu, m = _sizes(net)
    nth = net.n_bus - 1
    x = np.empty((ns, nx))
    x[:, :nth] = rng.normal(0.0, 0.05, (ns, nth))
    x[:, nth:] = rng.uniform(0.97, 1.03, (ns, nx - nth))
    hi = np.delete(net.pmax, net.gref)
    n = rng.standard_normal
    return dict(x=x, u=np.concatenate([rng.uniform(0.97, 1.03, net.n_gen),
                                       hi * rng.uniform(0.1, 0.9, net.n_gen - 1)]),
                y=n((ns, nx)) * (0.02 / ns), z=n((ns, m)) * (0.02 / ns),
                obj_weight=float(rng.uniform(1e-5, 4e-5)) / ns,
                sigma_x=rng.uniform(0.1, 10.0, (ns, nx)), sigma_u=rng.uniform(0.1, 10.0, nu),
                sigma_s=rng.uniform(0.1, 10.0, (ns, m)), r1x=n((ns, nx)), r1u=n(nu), r2=n((ns, m)),
                r3=n((ns, nx)), r4=n((ns, m)))


def _inputs(c, seed):
    """[(grid, active loads, reactive loads, iterate)] of a pass."""
    out = []
    for j, (net, ns) in enumerate(_grids(c)):
        rng = np.random.default_rng([seed, j])
        out.append((net, *_loads(net, ns, rng), _iterate(net, ns, rng)))
    return out


def _mlp_inputs(c, seed):
    g = torch.Generator().manual_seed(seed)
    sizes = [c["inputs"], c["hidden"], c["hidden"], c["hidden"], c["outputs"]]
    parts = []
    for fi, fo in zip(sizes[:-1], sizes[1:]):
        parts += [(torch.rand(fi * fo, generator=g) * 2 - 1) * (math.sqrt(6.0 / fi) / 2.0),
                  torch.randn(fo, generator=g) * 0.1]
    x = torch.randn(c["batch"], sizes[0], generator=g)
    t = torch.randn(c["batch"], sizes[-1], generator=g)
    return sizes, torch.cat(parts), x, t


def prepare(case, seed):
    if case["kind"] in ("forward", "train"):
        sizes, params, x, t = _mlp_inputs(case, seed)
        m = R.Mlp(sizes, case["batch"])
        m.set_params(params.cuda())
        return dict(case=case, mlp=m, x=x.cuda(), t=t.cuda(), y=torch.empty_like(t, device="cuda"),
                    grads=torch.zeros(m.n_params, device="cuda"), loss=torch.zeros(1, device="cuda"))
    if case["kind"] == "solve":
        net, ns = _grids(case)[0]
        pd, qd = _loads(net, ns, np.random.default_rng([seed, 0]), case["sigma"])
        p = R.rkkt_create(net, pd, qd)
        nx, nu, m = _sizes(net)
        out = {k: torch.zeros(n, dtype=F64, device="cuda")
               for k, n in dict(x=(ns, nx), u=nu, y=(ns, nx), z=(ns, m), s=(ns, m)).items()}
        return dict(case=case, handle=p, out=out)
    handles, its = [], []
    for net, pd, qd, it in _inputs(case, seed):
        ns, (nx, nu, m) = len(pd), _sizes(net)
        p = R.rkkt_create(net, pd, qd)
        a = {k: v if k == "obj_weight" else torch.tensor(v, dtype=F64, device="cuda") for k, v in it.items()}
        a["delta_w"] = case["delta_w"]
        for k, n in dict(f=ns, grad_x=(ns, nx), grad_u=(ns, nu), g=(ns, nx), h=(ns, m), khat=(nu, nu),
                         chol=(nu, nu), px=(ns, nx), pu=nu, ps=(ns, m), py=(ns, nx), pz=(ns, m)).items():
            a[k] = torch.zeros(n, dtype=F64, device="cuda")
        a["info"] = torch.zeros(1, dtype=torch.int32, device="cuda")
        handles.append(p)
        its.append(a)
    s = dict(case=case, handles=handles, its=its)
    torch.cuda.synchronize()
    if case["kind"] == "multi":
        s["multi"] = R.Multi(handles, its)
        if case["how"] == "graph":
            s["multi"].capture()
    elif case["how"] == "graph":
        R.rkkt_graph_capture(handles[0], its[0])
    return s


_OUT = ("f", "grad_x", "grad_u", "g", "h", "khat", "info", "px", "pu", "ps", "py", "pz")
_MULTI_OUT = ("khat", "px", "pu", "pz")  # of every grid: all of them would be over 64 outputs


def run(state):
    kind = state["case"]["kind"]
    if kind == "forward":
        state["mlp"].forward(state["x"], state["y"])
        return {"y": state["y"]}
    if kind == "train":
        m = state["mlp"]
        m.gradients(state["x"], state["t"], state["grads"], state["loss"])
        return {"grads": state["grads"], "loss": state["loss"]}
    if kind == "solve":
        r = R.rkkt_solve(state["handle"], **state["out"])
        return dict(state["out"], iters=int(r["iters"]), obj=float(r["obj"]))
    how, p, a = state["case"]["how"], state["handles"][0], state["its"][0]
    if kind == "multi":
        (state["multi"].launch if how == "graph" else state["multi"].iterate)()
        return [{k: b[k] for k in _MULTI_OUT} for b in state["its"]]
    if how == "graph":
        R.rkkt_graph_launch(p)
    elif how == "eager":
        R.rkkt_iterate(p, a)
    else:
        R.rkkt_evaluate(p, a["x"], a["u"], a["y"], a["z"], a["obj_weight"], a["f"], a["grad_x"], a["grad_u"],
                        a["g"], a["h"])
        R.rkkt_condense(p, a["sigma_x"], a["sigma_u"], a["sigma_s"], a["delta_w"], a["khat"])
        a["chol"].copy_(a["khat"])
        R.rkkt_factor(p, a["chol"], a["info"])
        R.rkkt_step(p, a["r1x"], a["r1u"], a["r2"], a["r3"], a["r4"], a["sigma_s"], a["chol"], a["px"],
                    a["pu"], a["ps"], a["py"], a["pz"])
    out = {k: a[k] for k in _OUT}
    if how == "calls":  # the caller's own factor (its upper triangle is not the factor's)
        out["chol"] = torch.tril(a["chol"])
    return out


def work(case):
    if case["kind"] in ("forward", "train"):
        h, b = case["hidden"], case["batch"]
        par = case["inputs"] * h + 2 * h * h + h * case["outputs"]
        if case["kind"] == "forward":
            return {"bytes": 4.0 * (par + b * (case["inputs"] + case["outputs"])), "flops": 2.0 * b * par}
        return {"bytes": 4.0 * (2 * par + b * (case["inputs"] + case["outputs"])), "flops": 6.0 * b * par}
    total = {"bytes": 0.0, "flops": 0.0}
    for net, ns in _grids(case):
        nx, nu, m = _sizes(net)
        links = net.n_bus + 2 * net.n_line         # nonzeros of a bus-by-bus matrix
        gx = 4.0 * links * (nx / (2.0 * net.n_bus)) ** 2
        # inputs and outputs of the four calls; multiply-adds of two forward
        # and two adjoint solves and one product per column on the patterns
        # without fill, of the scenario sum and the Cholesky
        by = 8.0 * (ns * (9 * nx + nu + 8 * m + 1) + 3 * nu * nu + 5 * nu)
        fl = ns * nu * (2 * 4 * gx + 2 * gx) + ns * nu * nu + nu ** 3 / 3.0
        k = 20 if case["kind"] == "solve" else 1   # about twenty iterations to a solution
        total["bytes"] += by if k == 1 else 8.0 * ns * (2 * nx + 2 * m + 2 * net.n_bus)
        total["flops"] += k * fl
    return total


# ------------------------------------------------- the same outputs, in 64 bits
def _second(c, th, v):
    """Second derivatives of Re sum_ik c_ik V_i conj(V_k) in (theta, v)."""
    d = c * torch.exp(1j * (th[:, None] - th[None, :]))
    q, r = d.real, -d.imag
    mm = v[:, None] * q * v[None, :]
    tt = mm + mm.T - torch.diag(mm.sum(1) + mm.sum(0))
    tv = torch.diag(r @ v - r.T @ v) + v[:, None] * (r - r.T)
    return torch.cat([torch.cat([tt, tv], 1), torch.cat([tv.T, q + q.T], 1)], 0)


class _Dense:
    """Dense model of one grid: power balance, flows and their derivatives."""

    def __init__(self, net, dev):
        t = lambda a: torch.as_tensor(np.asarray(a), device=dev)  # noqa: E731
        self.net, self.dev, self.nb = net, dev, net.n_bus
        self.f, self.t = t(net.line_from).long(), t(net.line_to).long()
        y = 1.0 / torch.complex(t(net.r), t(net.x))
        self.ys, self.sh = y, y + 0.5j * t(net.b)
        Y = torch.zeros(net.n_bus, net.n_bus, dtype=torch.complex128, device=dev)
        for a, b, w in ((self.f, self.f, self.sh), (self.t, self.t, self.sh), (self.f, self.t, -y),
                        (self.t, self.f, -y)):
            Y.index_put_((a, b), w, accumulate=True)
        self.Y = Y
        self.gb = t(net.gen_bus).long()
        bus = torch.arange(net.n_bus, device=dev)
        self.nonref = bus[bus != net.ref_bus]
        self.pq = bus[~torch.isin(bus, self.gb)]
        self.xc = torch.cat([self.nonref, self.nb + self.pq])
        self.uc = self.nb + self.gb
        self.gnr = torch.arange(net.n_gen, device=dev)
        self.gnr = self.gnr[self.gnr != net.gref]
        self.a, self.b, self.c0 = 1e4 * t(net.c2), 1e2 * t(net.c1), t(net.c0)

    def scenario(self, x, u, pd, qd, y, z, w):
        net, nb, dev = self.net, self.nb, self.dev
        ng, nl, ref = net.n_gen, net.n_line, net.ref_bus
        th, v = torch.zeros(nb, dtype=F64, device=dev), torch.zeros(nb, dtype=F64, device=dev)
        th[self.nonref], v[self.pq], v[self.gb] = x[:nb - 1], x[nb - 1:], u[:ng]
        pg = u[ng:]
        Pd, Qd = torch.zeros_like(th), torch.zeros_like(th)
        lb = torch.as_tensor(net.load_bus, device=dev).long()
        Pd[lb], Qd[lb] = pd, qd
        E = torch.exp(1j * th)
        V = v * E
        cur = self.Y @ V
        S = V * cur.conj()
        pgb = torch.zeros_like(th)
        pgb[self.gb[self.gnr]] = pg
        g = torch.cat([(S.real - pgb + Pd)[self.nonref], (S.imag + Qd)[self.pq]])
        pref = S.real[ref] + Pd[ref]
        Jth = 1j * V[:, None] * (torch.diag(cur) - self.Y * V[None, :]).conj()
        Jv = V[:, None] * (self.Y * E[None, :]).conj() + torch.diag(cur.conj() * E)
        J = torch.cat([Jth, Jv], 1)
        # line ends: S_a = V_a conj(sh V_a - ys V_b); derivatives in (th_a, th_b, v_a, v_b)
        ends, rows, c2 = [], [], torch.zeros(nb, nb, dtype=torch.complex128, device=dev)
        hess = torch.zeros(2 * nb, 2 * nb, dtype=F64, device=dev)
        for e, (a, b) in enumerate(((self.f, self.t), (self.t, self.f))):
            Va, Vb, Ea, Eb = V[a], V[b], E[a], E[b]
            Ia = self.sh * Va - self.ys * Vb
            Sa = Va * Ia.conj()
            d = torch.stack([1j * (Sa - Va * (self.sh * Va).conj()), -1j * Va * (-self.ys * Vb).conj(),
                             Ea * Ia.conj() + Va * (self.sh * Ea).conj(), Va * (-self.ys * Eb).conj()], 1)
            loc = torch.stack([a, b, nb + a, nb + b], 1)
            row = torch.zeros(nl, 2 * nb, dtype=F64, device=dev)
            row.scatter_(1, loc, 2 * (Sa.real[:, None] * d.real + Sa.imag[:, None] * d.imag))
            rows.append(row)
            ends.append(Sa.real ** 2 + Sa.imag ** 2)
            zz = z[1 + ng + e * nl:1 + ng + (e + 1) * nl]
            wt = 2 * zz * Sa.conj()
            c2.index_put_((a, a), wt * self.sh.conj(), accumulate=True)
            c2.index_put_((a, b), wt * (-self.ys).conj(), accumulate=True)
            blk = 2 * zz[:, None, None] * (d.real[:, :, None] * d.real[:, None, :]
                                           + d.imag[:, :, None] * d.imag[:, None, :])
            hess.index_put_((loc[:, :, None].expand(-1, 4, 4), loc[:, None, :].expand(-1, 4, 4)), blk,
                            accumulate=True)
        h = torch.cat([pref[None], (S.imag + Qd)[self.gb], *ends])
        cost = torch.zeros(ng, dtype=F64, device=dev)
        cost[self.gnr] = pg
        cost[net.gref] = pref
        f = w * (self.a * cost ** 2 + self.b * cost + self.c0).sum()
        dref = w * (2 * self.a[net.gref] * pref + self.b[net.gref])
        Jg = torch.cat([J.real[self.nonref], J.imag[self.pq]], 0)
        Jh = torch.cat([J.real[ref][None], J.imag[self.gb], *rows], 0)
        npg = ng - 1
        gu_pg = torch.zeros(len(self.xc), npg, dtype=F64, device=dev)
        pos = torch.full((nb,), -1, dtype=torch.long, device=dev)
        pos[self.nonref] = torch.arange(nb - 1, device=dev)
        gu_pg[pos[self.gb[self.gnr]], torch.arange(npg, device=dev)] = -1.0
        grad = dref * J.real[ref]
        gradu = torch.cat([grad[self.uc], w * (2 * self.a[self.gnr] * pg + self.b[self.gnr])])
        wp, wq = torch.zeros_like(th), torch.zeros_like(th)
        wp[self.nonref], wq[self.pq] = y[:nb - 1], y[nb - 1:]
        wp[ref] += z[0] + dref
        wq[self.gb] += z[1:1 + ng]
        hess += _second((wp - 1j * wq)[:, None] * self.Y.conj() + c2, th, v)
        hess += 2 * w * self.a[net.gref] * torch.outer(J.real[ref], J.real[ref])
        return SimpleNamespace(f=f, g=g, h=h, grad_x=grad[self.xc], grad_u=gradu, Gx=Jg[:, self.xc],
                               Gu=torch.cat([Jg[:, self.uc], gu_pg], 1), Hx=Jh[:, self.xc], Hv=Jh[:, self.uc],
                               Wxx=hess[self.xc][:, self.xc], Wxv=hess[self.xc][:, self.uc],
                               Wvv=hess[self.uc][:, self.uc], wpg=2 * w * self.a[self.gnr])


def _exact_pass(net, pd, qd, it, dw, dev):
    d = _Dense(net, dev)
    t = lambda a: torch.as_tensor(a, dtype=F64, device=dev)  # noqa: E731
    it = {k: v if k == "obj_weight" else t(v) for k, v in it.items()}
    pd, qd, ng = t(pd), t(qd), net.n_gen
    nx, nu, _ = _sizes(net)
    khat = torch.diag(it["sigma_u"] + dw)
    rhs = -it["r1u"]
    kept, out = [], {k: [] for k in ("f", "grad_x", "grad_u", "g", "h", "px", "ps", "py", "pz")}
    for k in range(len(pd)):
        s = d.scenario(it["x"][k], it["u"], pd[k], qd[k], it["y"][k], it["z"][k], it["obj_weight"])
        for n in ("f", "grad_x", "grad_u", "g", "h"):
            out[n].append(getattr(s, n))
        ss, r2, r4 = it["sigma_s"][k], it["r2"][k], it["r4"][k]
        kxx = s.Wxx + s.Hx.T @ (ss[:, None] * s.Hx) + torch.diag(it["sigma_x"][k] + dw)
        kxu, kuu = torch.zeros(nx, nu, dtype=F64, device=dev), torch.zeros(nu, nu, dtype=F64, device=dev)
        kxu[:, :ng] = s.Wxv + s.Hx.T @ (ss[:, None] * s.Hv)
        kuu[:ng, :ng] = s.Wvv + s.Hv.T @ (ss[:, None] * s.Hv)
        kuu[range(ng, nu), range(ng, nu)] = s.wpg
        sol = torch.linalg.solve(s.Gx, torch.cat([s.Gu, it["r3"][k][:, None]], 1))
        T, q = -sol[:, :nu], sol[:, nu]
        kt = kxx @ T + kxu
        khat = khat + T.T @ kt + kxu.T @ T + kuu
        wv = ss * r4 - r2
        r1 = it["r1x"][k] + s.Hx.T @ wv
        rhs = rhs - T.T @ (r1 - kxx @ q) + kxu.T @ q
        rhs[:ng] -= s.Hv.T @ wv
        if len(pd) * nx * nx * 8 > 4e9:   # kept for the recovery only where that fits
            s = None
        kept.append((s, kxx, kxu, T, q, r1, ss, r2, r4) if s is not None else (k, T, q, r1, ss, r2, r4))
    chol = torch.linalg.cholesky(khat)
    pu = torch.cholesky_solve(rhs[:, None], chol)[:, 0]
    for e in kept:
        if len(e) == 7:
            k, T, q, r1, ss, r2, r4 = e
            s = d.scenario(it["x"][k], it["u"], pd[k], qd[k], it["y"][k], it["z"][k], it["obj_weight"])
            kxx = s.Wxx + s.Hx.T @ (ss[:, None] * s.Hx) + torch.diag(it["sigma_x"][k] + dw)
            kxu = torch.zeros(nx, nu, dtype=F64, device=dev)
            kxu[:, :ng] = s.Wxv + s.Hx.T @ (ss[:, None] * s.Hv)
        else:
            s, kxx, kxu, T, q, r1, ss, r2, r4 = e
        px = T @ pu - q
        hp = s.Hx @ px + s.Hv @ pu[:ng]
        out["px"].append(px)
        out["py"].append(torch.linalg.solve(s.Gx.T, -(r1 + kxx @ px + kxu @ pu)))
        out["ps"].append(-(r4 + hp))
        out["pz"].append(ss * (hp + r4) - r2)
    res = {k: torch.stack(v) for k, v in out.items()}
    return dict(res, khat=khat, chol=chol, pu=pu, info=torch.zeros(1, dtype=torch.int32, device=dev))


def _gelu(a):
    return 0.5 * a * (1.0 + torch.erf(a / math.sqrt(2.0)))


def exact(case, seed):
    dev = "cuda" if torch.cuda.is_available() else "cpu"
    if case["kind"] in ("forward", "train"):
        sizes, params, x, t = _mlp_inputs(case, seed)
        p = params.double().to(dev).requires_grad_()
        a, off = x.double().to(dev), 0
        for l, (fi, fo) in enumerate(zip(sizes[:-1], sizes[1:])):
            a = a @ p[off:off + fi * fo].view(fi, fo) + p[off + fi * fo:off + fi * fo + fo]
            a = _gelu(a) if l < len(sizes) - 2 else a
            off += fi * fo + fo
        if case["kind"] == "forward":
            return {"y": a.detach()}
        loss = 0.5 * ((a - t.double().to(dev)) ** 2).sum() / x.shape[0]
        loss.backward()
        return {"grads": p.grad, "loss": loss.detach()[None]}
    if case["kind"] == "solve":
        return None   # an iterative solve: its end is known to the tolerance only
    if sum(ns * (net.n_bus / 1000.0) ** 3 for net, ns in _grids(case)) > 250.0:
        return None   # dense algebra that takes minutes
    got = [_exact_pass(*one, case["delta_w"], dev) for one in _inputs(case, seed)]
    if case["kind"] == "multi":
        return [{k: g[k] for k in _MULTI_OUT} for g in got]
    return {k: got[0][k] for k in _OUT + (("chol",) if case["how"] == "calls" else ())}
