"""The grid of the team kernels (csrc/rbd_team_plan.hpp, team_grid), on the CPU: at every accepted batch, up
to the largest of 2^30 instances, it stays within what one launch may hold (less than 2^32 lanes along an
axis) and its blocks start at instances of the batch, each 64 instances once."""
from __future__ import annotations

import shutil
import subprocess

import pytest

from paper_2604_04310_amd import build as B

MAIN = r"""
#include <cstdio>
#include <cstdlib>
#include "rbd_team_plan.hpp"
int main(int argc, char** argv) {
  const rbd::TeamGrid g = rbd::team_grid(std::atoll(argv[1]), std::atoi(argv[2]));
  std::printf("%u %u %u\n", g.x, g.y, rbd::kTeamRowBlocks);
}
"""


@pytest.fixture(scope="module")
def exe(tmp_path_factory):
    cxx = shutil.which("g++")
    if cxx is None:
        pytest.skip("no C++ compiler")
    d = tmp_path_factory.mktemp("grid")
    (d / "grid.cpp").write_text(MAIN)
    subprocess.run([cxx, "-std=c++17", "-Wall", "-Werror", f"-I{B.CSRC}", str(d / "grid.cpp"), "-o", str(d / "grid")],
                   check=True)
    return str(d / "grid")


@pytest.mark.parametrize("waves", [2, 3, 4])
@pytest.mark.parametrize("batch", [1, 64, 65, 65536, (1 << 29) + 1, (1 << 30) - 64, (1 << 30) - 63, 1 << 30])
def test_grid_holds_every_batch(exe, batch, waves):
    x, y, row = map(int, subprocess.run([exe, str(batch), str(waves)], capture_output=True, text=True,
                                        check=True).stdout.split())
    blocks = -(-batch // 64)
    assert x * waves * 64 < 1 << 32 and 1 <= y <= 65535
    # block (bx, by) starts at instance 64 (by row + bx)
    assert y == 1 or x == row
    assert x * y == blocks and (y - 1) * row + x == blocks
