"""The reduction on the elimination tree (variant 1 with 64-column tiles and
pull-form solves off chip, forced here on small grids) against the oracle:
one node and many, interface rows and control columns that fill strips
exactly or not at all, a hub bus whose node has many children, a reference bus
that splits the tree into a forest, odd scenario counts, and a grid whose
product takes 64 x 64 outputs per wavefront.  Reduced matrix 1e-10 (relative
Frobenius), every Newton-step block within gpu_common.step_bar; eager, graph
and repeated passes are equal bit for bit."""
import dataclasses

import numpy as np
import pytest

import gpu_common as gc
import synthgrid as sg

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

TREE = dict(variant=1, col_tile=64, sweep_form=2)


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


def _hub(n_arm, seed):
    """Arms of three buses around one bus, a generator at the hub's first arm
    end (the reference) and at every fourth arm end."""
    base = sg.make_network(3 * n_arm + 1, 3 * n_arm, 1 + n_arm // 4, seed, loads=n_arm)
    f, t = [], []
    for a in range(n_arm):
        f += [0, 1 + 3 * a, 2 + 3 * a]
        t += [1 + 3 * a, 2 + 3 * a, 3 + 3 * a]
    gen = np.array(sorted({3} | {3 * a for a in range(4, n_arm + 1, 4)}), dtype=np.int32)
    gen = gen[:base.n_gen]
    k = len(gen)
    return dataclasses.replace(
        base, n_gen=k, gen_bus=gen, ref_bus=int(gen[0]), line_from=np.array(f, dtype=np.int32),
        line_to=np.array(t, dtype=np.int32), pmin=base.pmin[:k], pmax=base.pmax[:k], qmin=base.qmin[:k],
        qmax=base.qmax[:k], c2=base.c2[:k], c1=base.c1[:k], c0=base.c0[:k])


def _split(seed):
    """Two grids that meet only at the reference bus."""
    a = sg.make_network(40, 56, 6, seed)
    nb = 79
    other = lambda b: np.where(b == a.ref_bus, a.ref_bus, np.where(b < a.ref_bus, b + 40, b + 39))  # noqa: E731
    gen2 = [int(other(b)) for b in a.gen_bus if b != a.ref_bus]
    order = np.argsort(np.concatenate([a.gen_bus, gen2]))
    cat = lambda v: np.concatenate([v, np.delete(v, a.ref_gen)])[order]  # noqa: E731
    return dataclasses.replace(
        a, n_bus=nb, n_line=112, n_gen=11, line_from=np.concatenate([a.line_from, other(a.line_from)]).astype(np.int32),
        line_to=np.concatenate([a.line_to, other(a.line_to)]).astype(np.int32), r=np.tile(a.r, 2), x=np.tile(a.x, 2),
        b=np.tile(a.b, 2), rate=np.tile(a.rate, 2),
        gen_bus=np.concatenate([a.gen_bus, gen2])[order].astype(np.int32), pmin=cat(a.pmin), pmax=cat(a.pmax),
        qmin=cat(a.qmin), qmax=cat(a.qmax), c2=cat(a.c2), c1=cat(a.c1), c0=cat(a.c0), vmin=np.full(nb, 0.9),
        vmax=np.full(nb, 1.1))


def _net(case):
    if case[0] == "hub":
        return _hub(case[1], 7)
    if case[0] == "split":
        return _split(11)
    return sg.make_network(*case)


CASES = [((2, 1, 1, 5), 3), ((5, 6, 2, 6), 2), ((9, 9, 8, 8), 1), ((17, 24, 8, 9), 5), ((60, 90, 33, 10), 7),
         (("hub", 40), 3), (("split",), 2), ((150, 220, 64, 12), 3), ((211, 300, 20, 13), 17),
         ((333, 500, 150, 14), 2), ((520, 760, 280, 15), 1)]


@pytest.mark.parametrize("case", CASES, ids=lambda c: f"{'-'.join(map(str, c[0]))}-N{c[1]}")
def test_tree_matches_the_oracle(case):
    net = _net(case[0])
    inst = sg.Instance("tree", net, sg.make_scenarios(net, case[1], 0.1, 5))
    it = gc.iterate(inst, seed=31)
    prob, ev, dg, red, dw = gc.oracle_state(inst, it)
    run = gc.GpuRun(inst, it, dw, torch, **TREE)
    run.evaluate()
    run.condense()
    run.factor()
    run.step()
    torch.cuda.synchronize()
    assert run.R.rkkt_status(run.p)[0] == 0
    kh = run.khat.cpu().numpy()
    assert np.array_equal(kh, kh.T)
    e_k = gc.rel_fro(kh, red.khat)
    print(f"\n  khat {e_k:.2e}", flush=True)
    assert e_k <= 1e-10
    st = gc.oracle_step(prob, ev, dg, red, dw, it)
    gc.check_step({k: v.cpu().numpy() for k, v in run.out.items()}, st, gc.cond2(red.khat))
    # the pass in one call, as a graph and again
    first = {k: v.clone() for k, v in run.out.items()}
    run.chol = torch.zeros_like(run.khat)
    args = gc.iter_args(run)
    run.R.rkkt_graph_capture(run.p, args)
    for rep in range(4):
        for v in run.out.values():
            v.fill_(float("nan"))
        run.khat.fill_(float("nan"))
        torch.cuda.synchronize()
        if rep == 0:
            run.R.rkkt_iterate(run.p, args)
        else:
            run.R.rkkt_graph_launch(run.p)
        torch.cuda.synchronize()
        assert np.array_equal(run.khat.cpu().numpy(), kh), rep
        assert all(torch.equal(run.out[k], first[k]) for k in first), rep


def test_tree_flags_singular_state_jacobians():
    """All magnitudes zero: every pivot is zero (the scenario that raised it is
    reported); the next pass on a regular point is clean."""
    net = sg.make_network(60, 90, 10, 3)
    inst = sg.Instance("tree", net, sg.make_scenarios(net, 2, 0.1, 5))
    it = gc.iterate(inst, seed=5)
    bad = dict(it, x=it["x"].copy(), u=it["u"].copy())
    bad["x"][:, net.n_bus - 1:] = 0.0
    bad["u"][:net.n_gen] = 0.0
    run = gc.GpuRun(inst, bad, 1.0, torch, **TREE)
    run.evaluate()
    run.condense()
    code, scen = run.R.rkkt_status(run.p)
    assert code == -3 and scen in (0, 1)
    run.inp["x"].copy_(gc.dev(it["x"], torch))
    run.inp["u"].copy_(gc.dev(it["u"], torch))
    run.evaluate()
    run.condense()
    assert run.R.rkkt_status(run.p)[0] == 0
    assert bool(torch.isfinite(run.khat).all())
