"""Up to which batch a tree's team runs an operation (csrc/rbd_team_plan.hpp, team_limit): on the CPU, that a
team with a longer chain never runs further than one with a shorter chain; on the GPU, both sides of the limits
(the kernels of a team and those of one instance per lane) against the oracle."""
from __future__ import annotations

import shutil
import subprocess

import pytest

import workloads as W
from paper_2604_04310_amd import build as B
from tests._models import TREE12

MAIN = r"""
#include <cstdio>
#include <initializer_list>
#include "rbd_team_plan.hpp"
int main() {
  using rbd::TeamOp;
  for (int nv : {17, 18, 24, 25, 35, 69})
    for (int waves = 0; waves <= rbd::kTeamWaves; ++waves)
      for (int trunk : {0, 3})
        for (int op = 0; op <= (int)TeamOp::kIdVjpExt; ++op) {
          for (int chain = 25; chain <= 75; ++chain) {
            rbd::TeamPlan p;
            p.waves = waves;
            p.chain = chain;
            p.trunk = trunk;
            std::printf("%lld ", rbd::team_limit(p, nv, (TeamOp)op));
          }
          std::printf("%d\n", waves);
        }
}
"""


def test_limits_fall_with_the_chain(tmp_path):
    cxx = shutil.which("g++")
    if cxx is None:
        pytest.skip("no C++ compiler")
    (tmp_path / "limits.cpp").write_text(MAIN)
    exe = str(tmp_path / "limits")
    subprocess.run([cxx, "-std=c++17", "-Wall", "-Werror", f"-I{B.CSRC}", str(tmp_path / "limits.cpp"), "-o", exe],
                   check=True)
    rows = [[int(x) for x in r.split()] for r in subprocess.run([exe], capture_output=True, text=True,
                                                                check=True).stdout.splitlines()]
    assert len(rows) == 6 * 5 * 2 * 10
    for *limits, waves in rows:
        if waves < 2:
            assert set(limits) == {0}
            continue
        assert all(a >= b for a, b in zip(limits, limits[1:]))
        assert min(limits) >= 16384 and max(limits) <= 1 << 30
        assert limits[-1] == 16384  # a chain of three quarters: one team per compute unit
        assert waves > 2 or set(limits) == {16384}


@pytest.fixture(scope="module")
def rbd():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2604_04310_amd as rbd
    rbd.lib()
    return rbd


ALL = ("fd", "rnea", "vjp", "rnea_vjp", "jvp", "rnea_jvp")
TREES = {"tree12f": (True, TREE12), "humanoid30": (True, W.humanoid().parent), **B.PREBUILT}


@pytest.mark.gpu
@pytest.mark.parametrize("name,limit,ops", [("arms18f", 16384, ALL), ("tree12f", 32768, ALL),
                                            ("arms25", 98304, ("rnea_vjp", "rnea_jvp")),
                                            ("tree20", 32768, ("vjp", "rnea_vjp")), ("tree20", 98304, ("fd",)),
                                            ("humanoid30", 98304, ("rnea_jvp",))])
@pytest.mark.parametrize("over", [0, 1])
def test_both_sides_of_a_limit(rbd, name, limit, ops, over):
    from tests.test_gpu_team import check_all
    fl, par = TREES[name]
    batch = limit + over
    desc = W.random_tree(list(par), fl, 870, rotated=True, gravity=W.tilted_gravity(871))
    sample = [0, 1, 63, 64, 127, batch // 2, batch - 66, batch - 65, batch - 2, batch - 1]
    check_all(rbd, rbd.Model(desc, 0), desc, batch, 872, ops, sample)
