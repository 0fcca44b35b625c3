"""Launch shapes of the blocked Cholesky (layout.h) on the host, up to orders whose
square does not fit 32 bits."""
import subprocess

from paper_2301_04869_amd import build as b

PROGRAM = """
#include <cstdio>
#include "layout.h"
int main() {
  for (int n : {129, 724, 725, 2889, 46340, 46341, 65535, 65536, 100000})
    std::printf("%d %d %d\\n", n, rkkt::chol_tiles(n), rkkt::chol_first_blocks(n));
}
"""


def test_first_launch_copies_large_matrices(tmp_path):
    src, exe = tmp_path / "shapes.cpp", str(tmp_path / "shapes")
    src.write_text(PROGRAM)
    subprocess.run([b.HIPCC, *b.COMMON, "-c", str(src), "-o", exe + ".o"], check=True, stderr=subprocess.DEVNULL)
    subprocess.run(["g++", exe + ".o", "-o", exe], check=True)
    out = subprocess.run([exe], check=True, stdout=subprocess.PIPE, text=True).stdout
    rows = [tuple(map(int, line.split())) for line in out.splitlines()]
    assert len(rows) == 9
    for n, tiles, blocks in rows:
        assert tiles == -(-n // 64)
        # one workgroup for the first tile, one per 1024 elements, at most 512
        assert blocks == 1 + min(512, -(-n * n // 1024)), n
