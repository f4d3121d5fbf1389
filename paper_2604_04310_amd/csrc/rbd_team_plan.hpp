// How the bodies of one tree are shared out over the waves of a team: several
// waves that work on the same 64 instances, each on its own branches. Host and
// device evaluate the same function (the device at compile time).
#pragma once

namespace rbd {

constexpr int kTeamWaves = 4;     // most waves of a team: one per SIMD of a compute unit
constexpr int kTeamMinDofs = 16;  // smaller trees stay one instance per lane
// Above this many DoFs a lane that does the whole tree holds more than the 256
// registers that two waves per SIMD leave it, and a team is faster at every
// batch (humanoid forward dynamics, team against one lane: 12 / 34 us at 4096,
// 26 / 39 at 65536, 48 / 88 at 131072); up to it some operations are faster one
// instance per lane once the batch fills the SIMDs (quadruped, 18 DoFs, forward
// dynamics: 14 / 15 us at 81920, 20 / 16 at 131072).
constexpr int kTeamAlwaysDofs = 24;
// Most rows of LDS (64 lanes, 256 bytes each) that a block of a team uses: two
// blocks share the 160 KB of a compute unit. What a trunk costs grows with its
// length and with the branches along it (the humanoid's four bodies: 319).
constexpr int kTeamRows = 320;

// The trunk is an ancestor-closed set of bodies; what hangs on it are the
// branches (whole subtrees). Every branch belongs to one wave; the trunk's own
// work, which needs all of its branches' results, is done by the owner.
struct TeamPlan {
  int waves = 0;               // 0: the tree does not split well enough
  int owner = 0;               // the wave that does the trunk's work (the one with the least of its own)
  signed char wave[64] = {};   // wave of a body, -1: trunk
  // waves whose branches are copies of each other (the same tree a constant
  // number of bodies later, on the same trunk bodies) run the same code: that
  // of wave role[w], with body indices moved by shift[w]
  int role[kTeamWaves] = {};
  int shift[kTeamWaves] = {};
};

// Starts from the roots as branches and keeps moving the root of the largest
// branch into the trunk; every such trunk is rated by its longest chain of
// work, in tenths of a body: a wave's own branches (10 a body) and the trunk
// bodies above them that it runs down again (2), then the trunk (10 a body),
// which the other waves wait for. Branches go to waves largest first, each to
// the least loaded wave. The best trunk is taken if that chain is at most
// three quarters of the whole tree's work. Trunks whose waves hand over more than
// kTeamRows in any operation are left out.
constexpr TeamPlan team_plan(bool floating, int n, const int* parent) {
  TeamPlan best;
  int size[64] = {}, dofs[64] = {}, above_dofs[64] = {}, nv = 0;
  for (int i = 0; i < n; ++i) {
    dofs[i] = floating && i == 0 ? 6 : 1;
    above_dofs[i] = parent[i] < 0 ? 0 : above_dofs[parent[i]] + dofs[parent[i]];
    nv += dofs[i];
  }
  for (int i = n - 1; i >= 0; --i) {
    size[i] += 1;
    if (parent[i] >= 0) size[parent[i]] += size[i];
  }
  bool trunk[64] = {};
  int br[64] = {};
  int nb = 0, nt = 0, best_cost = 0;
  for (int i = 0; i < n; ++i)
    if (parent[i] < 0) br[nb++] = i;
  for (;;) {
    // the largest branch first (stable)
    for (int a = 1; a < nb; ++a)
      for (int c = a; c > 0 && size[br[c]] > size[br[c - 1]]; --c) {
        const int x = br[c];
        br[c] = br[c - 1];
        br[c - 1] = x;
      }
    if (nb > 1 && (!floating || trunk[0])) {
      int load[kTeamWaves] = {}, wave[64] = {};
      for (int k = 0; k < nb; ++k) {
        int w = 0;
        for (int c = 1; c < kTeamWaves; ++c)
          if (load[c] < load[w]) w = c;
        load[w] += 10 * size[br[k]];
        wave[k] = w;
      }
      int longest = 0, owner = 0, least = 0, used = 0;
      int att = 0, schur = 0, rhs = 0, nvt = 0;  // over the waves: trunk bodies with branches, rows of the factor,
                                                 // DoFs above; DoFs of the trunk
      for (int w = 0; w < kTeamWaves; ++w) {
        bool above[64] = {}, holds[64] = {};
        int anc = 0;
        for (int k = 0; k < nb; ++k) {
          if (wave[k] != w) continue;
          const int on = parent[br[k]];
          if (on >= 0 && !holds[on]) {
            holds[on] = true;
            ++att;
          }
          for (int a = on; a >= 0 && !above[a]; a = parent[a]) {
            above[a] = true;
            anc += 2;
            for (int d = 0; d < dofs[a]; ++d) schur += above_dofs[a] + d + 1;
            rhs += dofs[a];
          }
        }
        if (load[w] == 0) continue;
        ++used;
        if (load[w] + anc > longest) longest = load[w] + anc;
        if (least == 0 || load[w] + anc < least) {
          least = load[w] + anc;
          owner = w;
        }
      }
      for (int i = 0; i < n; ++i) nvt += trunk[i] ? dofs[i] : 0;
      // the blocks' rows as the kernels count them: articulated-body form,
      // adjoint, tangent, operational-space control
      const int rows[] = {27 * att + 6 * nt,
                          16 * att + schur + 2 * rhs + 2 * nvt,
                          2 * nv + 30 * att + 2 * nvt,
                          16 * att + schur + rhs + nvt,
                          nv + 12 * att + rhs + nvt,
                          16 * att + schur + rhs + 6 * nvt + 39};
      bool fits = true;
      for (int r : rows) fits = fits && r <= kTeamRows;
      const int cost = longest + 10 * nt;
      if (fits && used > 1 && (best.waves == 0 || cost < best_cost)) {
        best_cost = cost;
        best.waves = used;  // waves 0 .. used - 1 have work
        best.owner = owner;
        for (int i = 0; i < n; ++i) best.wave[i] = -1;
        for (int k = 0; k < nb; ++k)
          for (int i = br[k]; i < br[k] + size[br[k]]; ++i) best.wave[i] = (signed char)wave[k];
      }
    }
    if (nb == 0 || size[br[0]] == 1 || nt >= n / 2 || nb > 16) break;
    int s = 0;
    if (floating && !trunk[0])
      while (br[s] != 0) ++s;
    const int b = br[s];
    trunk[b] = true;
    ++nt;
    for (int k = s; k + 1 < nb; ++k) br[k] = br[k + 1];
    --nb;
    for (int c = b + 1; c < b + size[b]; c += size[c]) br[nb++] = c;
  }
  if (best.waves == 0 || 4 * best_cost > 3 * 10 * n) return TeamPlan{};
  // copies: wave w's bodies are wave v's moved by d
  for (int w = 0; w < best.waves; ++w) {
    best.role[w] = w;
    for (int v = 0; v < w && best.role[w] == w; ++v) {
      if (best.role[v] != v) continue;
      int fv = 0, fw = 0;
      while (best.wave[fv] != v) ++fv;
      while (best.wave[fw] != w) ++fw;
      const int d = fw - fv;
      bool same = true;
      for (int i = 0; i < n && same; ++i) {
        const bool in_v = best.wave[i] == v;
        const bool in_w = i + d >= 0 && i + d < n && best.wave[i + d] == w;
        same = in_v == in_w;
        if (same && in_v) {
          const int p = parent[i], q = parent[i + d];
          same = (p < 0 || best.wave[p] < 0) ? q == p : q == p + d;
        }
      }
      // every body of w has its image (counts equal)
      int cv = 0, cw = 0;
      for (int i = 0; i < n; ++i) {
        cv += best.wave[i] == v;
        cw += best.wave[i] == w;
      }
      if (same && cv == cw) {
        best.role[w] = v;
        best.shift[w] = d;
      }
    }
  }
  return best;
}

// The grid of a team kernel, one block of waves * 64 lanes per 64 instances. A
// launch holds less than 2^32 lanes along an axis, which four waves reach at the
// largest batch (2^30: 2^24 blocks): that one goes out as two rows of blocks.
constexpr unsigned kTeamRowBlocks = 1u << 23;
struct TeamGrid {
  unsigned x, y;
};
constexpr TeamGrid team_grid(long long batch, int waves) {
  const unsigned long long blocks = (unsigned long long)(batch + 63) / 64;
  if (blocks * waves * 64 < (1ull << 32)) return {(unsigned)blocks, 1};
  return {kTeamRowBlocks, (unsigned)((blocks + kTeamRowBlocks - 1) / kTeamRowBlocks)};
}

}  // namespace rbd
