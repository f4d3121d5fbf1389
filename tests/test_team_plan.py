"""How a tree is shared out over a team of waves (csrc/rbd_team_plan.hpp), on the CPU: over random
depth-first trees every plan covers the tree with a trunk closed under ancestors and whole branches, the
owner is a wave of the team, and waves that share code have identical branches."""
from __future__ import annotations

import os
import shutil
import subprocess

import numpy as np
import pytest

import workloads as W
from paper_2604_04310_amd import build as B

MAIN = r"""
#include <cstdio>
#include "rbd_team_plan.hpp"
int main() {
  int f, n, p[64];
  while (std::scanf("%d %d", &f, &n) == 2) {
    for (int i = 0; i < n; ++i) if (std::scanf("%d", p + i) != 1) return 1;
    const rbd::TeamPlan t = rbd::team_plan(f != 0, n, p);
    std::printf("%d %d", t.waves, t.owner);
    for (int w = 0; w < rbd::kTeamWaves; ++w) std::printf(" %d %d", t.role[w], t.shift[w]);
    for (int i = 0; i < n; ++i) std::printf(" %d", t.wave[i]);
    std::printf("\n");
  }
}
"""


def plans(trees, tmp_path):
    cxx = shutil.which("g++")
    if cxx is None:
        pytest.skip("no C++ compiler")
    src = tmp_path / "plan.cpp"
    src.write_text(MAIN)
    exe = str(tmp_path / "plan")
    subprocess.run([cxx, "-std=c++17", "-O1", "-Wall", "-Werror", f"-I{B.CSRC}", str(src), "-o", exe], check=True)
    text = "".join(f"{int(f)} {len(p)} {' '.join(map(str, p))}\n" for f, p in trees)
    out = subprocess.run([exe], input=text, capture_output=True, text=True, check=True).stdout.splitlines()
    assert len(out) == len(trees)
    return [np.array(line.split(), int) for line in out]


def test_plans_of_random_trees(tmp_path):
    rng = np.random.default_rng(5)
    trees = [(f, p) for f, p in B.PREBUILT.values()] + [(f, p) for f, p in B.compiled_topologies().values()]
    for n in list(range(1, 65)) * 4:
        trees.append((bool(rng.integers(2)), [int(x) for x in W.random_dfs_parents(n, int(rng.integers(1 << 30)))]))
    teams = 0
    for (floating, par), t in zip(trees, plans(trees, tmp_path)):
        n, (waves, owner), roles, wave = len(par), t[:2], t[2:10].reshape(4, 2), t[10:]
        if waves == 0:
            continue
        teams += 1
        assert 2 <= waves <= 4 and 0 <= owner < waves
        assert set(wave) <= set(range(-1, waves)) and set(range(waves)) <= set(wave)
        assert not floating or wave[0] == -1
        for i, p in enumerate(par):
            if wave[i] < 0:
                assert p < 0 or wave[p] < 0  # the trunk is closed under ancestors
            else:
                assert p < 0 or wave[p] in (-1, wave[i])  # a branch is a whole subtree of one wave
        for w in range(waves):
            r, d = roles[w]
            assert roles[r][0] == r and roles[r][1] == 0
            mine, model = np.flatnonzero(wave == w), np.flatnonzero(wave == r)
            assert (mine == model + d).all()
            for i, j in zip(mine, model):
                pi, pj = par[i], par[j]
                assert pi == pj if pj < 0 or wave[pj] < 0 else pi == pj + d
    assert teams > 50
