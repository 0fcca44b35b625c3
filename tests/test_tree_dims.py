"""Which form the reduction takes is visible to the caller: rkkt_dims.tree, from the
host analysis, for automatic and forced shapes."""
import pytest

import paper_2301_04869_amd as R
import synthgrid as sg


def _analyze(net, n_scen, **opts):
    import ctypes
    s, keep = R._lib._host_network(net)
    o, d = R._lib.Options(), R._lib.Dims()
    for k, v in opts.items():
        setattr(o, k, v)
    assert R.lib().rkkt_analyze(ctypes.byref(s), n_scen, ctypes.byref(o), ctypes.byref(d)) == 0
    return d.as_dict()


@pytest.mark.parametrize("buses,opts,tree", [
    (118, {}, 0),                                            # fits on chip
    (300, {}, 1),
    (300, dict(variant=2), 0),                               # the stacked product
    (300, dict(variant=1, col_tile=32), 0),                  # another tile: panels
    (300, dict(variant=1, sweep_form=1), 0),                 # push form: panels
    (118, dict(variant=1, col_tile=64, sweep_form=2), 1)])
def test_dims_tell_the_tree(buses, opts, tree):
    net = sg.make_network(buses, int(1.5 * buses), buses // 3, 5)
    d = _analyze(net, 4, **opts)
    assert d["tree"] == tree
    if tree:
        assert (d["variant"], d["lds_reduce"], d["sweep_form"]) == (1, 0, 2)
