"""When the elimination tree is given up for its memory, on the host: where it takes
more than panels in device memory, the difference may be a sixteenth of what is
free; where it takes less, it is taken whatever is free."""
import os
import subprocess

import pytest

import synthgrid as sg
from paper_2301_04869_amd import build as b

HERE = os.path.dirname(os.path.abspath(__file__))


@pytest.fixture(scope="module")
def exe(tmp_path_factory):
    d = tmp_path_factory.mktemp("tree_memory")
    objs = []
    for src in (os.path.join(HERE, "tree_memory.cpp"), os.path.join(b.CSRC, "symbolic.cpp"),
                os.path.join(b.CSRC, "tree.cpp")):
        objs.append(str(d / (os.path.basename(src) + ".o")))
        subprocess.run([b.HIPCC, *b.COMMON, "-c", src, "-o", objs[-1]], check=True, stderr=subprocess.DEVNULL)
    subprocess.run(["g++", *objs, "-o", str(d / "tree_memory")], check=True)
    return str(d / "tree_memory")


def _bytes(exe, net, n_scen):
    lines = "\n".join(f"{f} {t}" for f, t in zip(net.line_from, net.line_to))
    inp = f"{net.n_bus} {net.n_line} {net.n_gen} {net.ref_bus} {n_scen}\n{lines}\n{' '.join(map(str, net.gen_bus))}\n"
    out = subprocess.run([exe], input=inp, check=True, stdout=subprocess.PIPE, text=True).stdout
    return tuple(map(int, out.split()))


@pytest.mark.parametrize("n_scen", [1, 16, 600])
def test_more_memory_than_panels(exe, n_scen):
    tree, panel, free = _bytes(exe, sg.make_network(200, 310, 50, 5), n_scen)
    assert tree > panel
    assert free == 16 * (tree - panel)


def test_less_memory_than_panels(exe):
    tree, panel, free = _bytes(exe, sg.make_network(2000, 3000, 300, 5), 8)
    assert tree < panel and free == 0
