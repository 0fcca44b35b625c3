"""A grid without load buses, made and used at once on a stream that does not wait
for the null stream: the pass equals that of the same grid with zero loads."""
import dataclasses

import numpy as np
import pytest

import gpu_common as gc
import synthgrid as sg

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


@pytest.mark.parametrize("opts", [{}, dict(variant=1, col_tile=64, sweep_form=2)], ids=["chip", "tree"])
def test_no_loads_equal_zero_loads(opts):
    net = sg.make_network(150, 220, 64, 12)
    zero = sg.Instance("zero", net, dataclasses.replace(sg.make_scenarios(net, 40, 0.1, 5)))
    zero.scen.pd[:] = 0.0
    zero.scen.qd[:] = 0.0
    none = np.zeros(0)
    bare = sg.Instance("none", dataclasses.replace(net, load_bus=none.astype(np.int32), pd=none, qd=none),
                       dataclasses.replace(zero.scen, pd=np.zeros((0, 40)), qd=np.zeros((0, 40))))
    it = gc.iterate(zero, seed=3)
    outs = []
    for inst in (zero, bare):
        with torch.cuda.stream(torch.cuda.Stream()):
            run = gc.GpuRun(inst, it, 1.0, torch, **opts)
            run.evaluate()
            run.condense()
            run.factor()
            run.step()
            torch.cuda.synchronize()
            assert run.R.rkkt_status(run.p)[0] == 0 and int(run.info.item()) == 0
        outs.append([run.g, run.h, run.khat, *run.out.values()])
    assert all(torch.equal(a, b) for a, b in zip(*outs))
