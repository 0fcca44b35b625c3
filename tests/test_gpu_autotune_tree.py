"""The autotuner on a grid whose fastest shape is the elimination tree: scenario
groups and chain rows, which the tree does not have, are not timed against each
other (their automatic values are returned), and the shape runs on the tree."""
import pytest

import synthgrid as sg

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


def test_tree_shapes_are_timed_once():
    import paper_2301_04869_amd as R
    net = sg.make_network(400, 600, 60, 5)
    scen = sg.make_scenarios(net, 4, 0.1, 6)
    for _ in range(3):
        opts, ms = R.rkkt_autotune(net, scen.pd.T, scen.qd.T, reps=2)
        print(f"\n  {opts} {ms:.3f} ms")
        p = R.rkkt_create(net, scen.pd.T, scen.qd.T, **opts)
        assert p.dims["tree"] == 1 and 0.0 < ms < 100.0
        assert opts["scen_per_group"] == 0 and opts["chain_rows"] == 0
