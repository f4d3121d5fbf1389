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


def comb(spine, rib):
    """A chain of `spine` bodies, each with a chain of `rib` bodies hanging on it."""
    par, last = [], -1
    for _ in range(spine):
        me = at = len(par)
        par.append(last)
        for _ in range(rib):
            par.append(at)
            at = len(par) - 1
        last = me
    return par


@pytest.mark.parametrize("floating", [False, True])
def test_rows_of_a_block_fit(tmp_path, floating):
    """Long trunks with branches all along hand over the most: the rows of LDS of the largest block (the
    adjoint's and operational-space control's) stay within the 320 that let two blocks share a compute unit."""
    trees = [(floating, comb(s, r)) for s in range(2, 32) for r in range(1, 64 // s)]
    rng = np.random.default_rng(6)
    trees += [(floating, [int(x) for x in W.random_dfs_parents(64, int(rng.integers(1 << 30)))]) for _ in range(200)]
    teams = 0
    for (_, par), t in zip(trees, plans(trees, tmp_path)):
        n, waves, wave = len(par), t[0], t[10:]
        if waves == 0:
            continue
        teams += 1
        dofs = [6 if floating and i == 0 else 1 for i in range(n)]
        depth = np.zeros(n, int)
        for i, p in enumerate(par):
            depth[i] = 0 if p < 0 else depth[p] + dofs[p]
        trunk_dofs = sum(d for d, w in zip(dofs, wave) if w < 0)
        att = factor = rhs = 0
        for w in range(waves):
            on = {par[i] for i in range(n) if wave[i] == w and par[i] >= 0 and wave[par[i]] < 0}
            att += len(on)
            above = set()
            for a in on:
                while a >= 0:
                    above.add(a)
                    a = par[a]
            factor += sum(depth[a] + d + 1 for a in above for d in range(dofs[a]))
            rhs += sum(dofs[a] for a in above)
        adjoint = max(16 * att + factor + 2 * rhs, 2 * sum(dofs) + 30 * att) + 2 * trunk_dofs
        control = 16 * att + factor + rhs + 6 * trunk_dofs + 39
        assert max(adjoint, control, 27 * att + 6 * int((wave < 0).sum())) <= 320
    assert teams > 50
