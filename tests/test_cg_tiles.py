"""How many nodes the CG kernels' blocks cover on strips (host arithmetic of
cg_mg.hpp, CPU only): a block's tile holds 512 nodes, and what it holds past the
edge of the grid is work for nothing."""
import os
import shutil
import subprocess

import pytest

from paper_1810_11685_amd import build as B

DRIVER = r"""
#include <cstdio>
#include <cstdlib>
#include "cg_mg.hpp"
int main(int argc, char** argv) {
  for (int i = 1; i + 1 < argc; i += 2) std::printf("%d\n", qpat::cgmg::tiles(std::atoi(argv[i]), std::atoi(argv[i + 1])));
}
"""


@pytest.mark.skipif(shutil.which("hipcc") is None and not os.path.exists("/opt/rocm/bin/hipcc"), reason="hipcc not found")
def test_tiles_of_strips_are_mostly_inside(tmp_path):
    (tmp_path / "tiles.hip").write_text(DRIVER)
    exe = str(tmp_path / "tiles")
    subprocess.run([B.hipcc(), *B.HIP_FLAGS, "-I", B.CSRC, str(tmp_path / "tiles.hip"), "-o", exe],
                   check=True)
    sizes = [(w, 2000) for w in range(2, 33)] + [(2000, h) for h in range(2, 33)]
    out = subprocess.run([exe, *(str(v) for s in sizes for v in s)], check=True, capture_output=True, text=True).stdout
    for (nx, ny), n in zip(sizes, map(int, out.split())):
        assert nx * ny <= 512 * n <= 3.5 * nx * ny, (nx, ny, n)
