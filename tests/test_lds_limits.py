"""Dynamic LDS limits (lds_limit.cpp) on the host, with a stand-in for the HIP
runtime: raised on every device that a handle is made on, never lowered, from
several threads."""
import os
import subprocess

from paper_2301_04869_amd import build as b

HERE = os.path.dirname(os.path.abspath(__file__))


def test_limits_per_device_and_thread(tmp_path):
    objs = []
    for src in (os.path.join(HERE, "lds_limits.cpp"), os.path.join(b.CSRC, "lds_limit.cpp")):
        objs.append(str(tmp_path / (os.path.basename(src) + ".o")))
        subprocess.run([b.HIPCC, *b.COMMON, "-O1", "-c", src, "-o", objs[-1]], check=True, stderr=subprocess.DEVNULL)
    exe = str(tmp_path / "lds_limits")
    subprocess.run(["g++", *objs, "-o", exe, "-pthread"], check=True)
    assert subprocess.run([exe], stdout=subprocess.PIPE, text=True, timeout=60).stdout.strip() == "ok"
