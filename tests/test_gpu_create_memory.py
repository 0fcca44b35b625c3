"""A handle whose elimination tree does not fit in the device's free memory is
made with panels in device memory instead, and computes the same."""
import pytest

import gpu_common as gc
import synthgrid as sg

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


def test_panels_where_the_tree_does_not_fit():
    import paper_2301_04869_amd as R
    net = sg.make_network(200, 310, 50, 5)
    scen = sg.make_scenarios(net, 600, 0.1, 6)
    inst = sg.Instance("memory", net, scen)
    run = gc.GpuRun(inst, gc.iterate(inst, seed=3), 1.0, torch)
    run.evaluate()
    run.condense()
    torch.cuda.synchronize()
    want = run.khat.cpu().numpy().copy()
    need = run.p.dims["workspace_bytes"]
    torch.cuda.empty_cache()
    get = lambda n: torch.empty(n, dtype=torch.uint8, device="cuda")  # noqa: E731
    held = [get(torch.cuda.mem_get_info()[0] - need * 4 // 5)]
    for _ in range(400):   # the device may give more than it reports as free
        try:
            get(need * 9 // 10)
        except torch.cuda.OutOfMemoryError:
            break
        torch.cuda.empty_cache()
        held.append(get(need // 16))
    torch.cuda.empty_cache()
    run.p = R.rkkt_create(net, scen.pd.T, scen.qd.T)
    assert run.p.dims["workspace_bytes"] < need * 4 // 5
    del held
    torch.cuda.empty_cache()
    run.khat.zero_()
    run.evaluate()
    run.condense()
    torch.cuda.synchronize()
    # two computations of one matrix in FP64, each within 1e-10 of the oracle
    assert gc.rel_fro(run.khat.cpu().numpy(), want) <= 2e-10
