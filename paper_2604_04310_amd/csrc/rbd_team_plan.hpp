// How the bodies of one tree are shared out over the waves of a team: several
// waves that work on the same 64 instances, each on its own branches. Host and
// device evaluate the same function (the device at compile time).
#pragma once

namespace rbd {

constexpr int kTeamWaves = 4;     // most waves of a team: one per SIMD of a compute unit
constexpr int kTeamMinDofs = 16;  // smaller trees stay one instance per lane
// Above this many DoFs a lane that does the whole tree holds more than the 256
// registers that two waves per SIMD leave it (see team_limit).
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
  int chain = 0;               // the longest chain of work, percent of the whole tree's (see team_plan)
  int trunk = 0;               // bodies of the trunk
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
// kTeamRows in any operation are left out, and those that leave one wave more
// than two thirds of the bodies: it holds about what a lane with the whole tree
// holds (27 bodies, 19 on one wave: adjoint and tangent of forward dynamics 64.6
// and 62.7 us at batch 16384 against 61.3 and 56.7 on one lane; 26 bodies, 17 on
// one: 47.8 and 51.3 against 54.2 and 52.9).
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
      int longest = 0, owner = 0, least = 0, used = 0, most = 0;
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
        if (load[w] > most) most = load[w];
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
      bool fits = 3 * most <= 2 * 10 * n;
      for (int r : rows) fits = fits && r <= kTeamRows;
      const int cost = longest + 10 * nt;
      if (fits && used > 1 && (best.waves == 0 || cost < best_cost)) {
        best_cost = cost;
        best.waves = used;  // waves 0 .. used - 1 have work
        best.owner = owner;
        best.chain = (100 * cost + 10 * n - 1) / (10 * n);
        best.trunk = nt;
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

// The operations that are shared out, by the batch up to which they are.
enum class TeamOp { kFd, kFdExt, kId, kVjp, kVjpExt, kJvp, kIdJvp, kIdJvpExt, kIdVjp, kIdVjpExt };
constexpr long long kTeamEvery = 1ll << 30;

// The largest batch at which a tree's team runs an operation; above it one
// instance per lane. 16384 instances are one team for every compute unit, each
// wave on a SIMD of its own; beyond that teams share the SIMDs, as many as their
// registers admit (one to three), while one instance per lane has SIMDs to spare
// up to 65536. So the shorter a team's chain, the later the other catches up.
// Measured against one lane, us (trees by DoFs and `chain`):
//   two waves, or a chain above 60: better up to 16384 everywhere. Tangent at
//     24576: 84.7/68.4 (36 DoFs, 66), 66.7/53.5 (31, 75), 44.9/48.0 (24, 75);
//     forward dynamics 11.3/10.1 at 32768 (18 DoFs, 54, two waves).
//   above 45: better up to 32768 (17 DoFs, 52: adjoint 16.9/22.4, with forces
//     36.1/36.0; 29, 47: tangent 42.7/47.4; 27, 52: 25.9/41.1), not above: 40000
//     25.4/23.8 and 52.5/44.9; 65536 90.6/82.6; forward dynamics 25.1/23.6 (23, 47).
//   up to 45, more than 24 DoFs: better at every batch (35 DoFs, 40, at 65536 and
//     393216: forward dynamics 27/42 and 128/228, adjoint 67/89 and 348/563,
//     tangent 66/111 and 381/669; 29, 43: 21/26 and 103/146, 47/63 and 260/376,
//     50/79 and 292/463), but
//     tangent of inverse dynamics (35, 40): 60/70 at 98304, 82/77 at 131072,
//       254/192 at 393216;
//     its adjoint with forces above 40: 39/57 at 32768, 73/61 at 65536 (29, 43;
//       35, 40: 82/97 and, at 393216, 530/619); with no trunk at all that and the
//       tangent with forces: 78/100 and 76/93 at 98304, 192/169 and 164/143 at 196608.
//   up to 45, 17 to 24 DoFs: 18 DoFs, 33, at 65600, 98304, 131072 and 262144:
//     forward dynamics 13.3/14.7, 16.3/15.5, 20.4/16.3, 37.0/31.0 (14.1/15.5 at 81920)
//       with forces    16.1/28.0, 20.0/30.4, 24.9/32.4, 45.2/58.1
//     its adjoint      23.8/31.9, 28.5/33.7, 36.6/34.3, 66.1/64.8
//     its tangent      22.6/37.1, 27.3/43.9, 35.0/47.8, 65.8/82.5
//     inverse dynamics  8.6/8.3,   8.9/8.7,   9.4/9.4,  17.7/18.0
//       (its kernel alone 6.9 at 81920; 9.0 at 98304 on one lane)
//       its adjoint    13.7/19.3, 18.5/22.4, 22.4/24.4, 38.4/44.1
//       its tangent    12.9/14.9, 16.9/19.6, 20.7/22.0, 37.1/35.7
//     and 20 DoFs, 42, with forces: forward dynamics 26/32 at 81920, 39/35 at
//     131072; its adjoint 45/103 at 32768, 85/79 at 65536.
// Where one operation turns later than another of the same line, the line is the
// earlier one's.
constexpr long long team_limit(const TeamPlan& p, int nv, TeamOp op) {
  if (p.waves < 2) return 0;
  if (p.waves == 2 || p.chain > 60) return 16384;
  if (p.chain > 45) return 32768;
  const bool uneven = p.chain > 40, bare = p.trunk == 0;
  if (op == TeamOp::kIdVjpExt) return uneven ? 32768 : (bare ? 98304 : kTeamEvery);
  if (op == TeamOp::kIdJvpExt) return bare ? 98304 : kTeamEvery;
  if (nv > kTeamAlwaysDofs) return op == TeamOp::kIdJvp ? 98304 : kTeamEvery;
  if (op == TeamOp::kFd || op == TeamOp::kId || op == TeamOp::kVjp || op == TeamOp::kIdJvp) return 81920;
  if (op == TeamOp::kVjpExt) return uneven ? 32768 : kTeamEvery;
  if (op == TeamOp::kFdExt) return uneven ? 98304 : kTeamEvery;
  return kTeamEvery;
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
