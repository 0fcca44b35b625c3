"""The interior-point driver's order of calls, on the host: ipm.cpp linked with
stand-ins that compute nothing (ipm_calls.cpp).  Every way out of a solve, those
after a failing runtime call included, leaves no work behind on the handle's
second stream, and residuals are formed from the iterate's values only."""
import os
import subprocess

import pytest

from paper_2301_04869_amd import build as b

HERE = os.path.dirname(os.path.abspath(__file__))


@pytest.fixture(scope="module")
def solves(tmp_path_factory):
    d = tmp_path_factory.mktemp("ipm_calls")
    objs = []
    for src in (os.path.join(HERE, "ipm_calls.cpp"), os.path.join(b.CSRC, "ipm.cpp")):
        objs.append(str(d / (os.path.basename(src) + ".o")))
        subprocess.run([b.HIPCC, *b.COMMON, "-O1", "-c", src, "-o", objs[-1]], check=True, stderr=subprocess.DEVNULL)
    exe = str(d / "ipm_calls")
    subprocess.run(["g++", *objs, "-o", exe], check=True)
    out = subprocess.run([exe], check=True, stdout=subprocess.PIPE, text=True, timeout=60).stdout
    return [tuple(map(int, line.split())) for line in out.splitlines()]


def test_every_exit_is_reached(solves):
    plain = {s[0]: s for s in solves if s[1] == 0}
    assert [plain[m][3] for m in range(4)] == [0, 2, 3, 4]   # converged, line search, inertia, device status
    assert all(s[2] == 0 for s in plain.values())
    assert sum(s[2] != 0 for s in solves) > 100               # failing runtime calls


def test_residuals_come_from_the_iterate(solves):
    assert [s for s in solves if s[2] == 0 and not s[5]] == []


def test_nothing_is_left_on_the_second_stream(solves):
    assert [s for s in solves if not s[4]] == []
