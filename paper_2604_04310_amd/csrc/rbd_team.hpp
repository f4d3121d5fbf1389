// A team of waves per 64 instances: lane l of every wave of a block works on
// the same instance, each wave on its own branches of the tree, and the wave
// that owns the trunk finishes it.
//
// One lane doing a whole tree is one serial chain: the humanoid's forward
// dynamics is 16 thousand vector instructions whatever the batch, and its
// registers admit one wave per SIMD, which then issues one instruction every
// 5.8 cycles. Split by branches, the chain is the longest branch, the trunk
// bodies above it and the trunk (118 tenths of a body of 300, rbd_team_plan.hpp),
// a batch fills four times as many waves, and a wave holds only what its own
// branches need, so two or three waves fit on a SIMD and hide each other's latency.
//
// The branches of different waves meet in the trunk only: what a branch hands
// over is the force and the (composite or articulated) inertia it exerts on the
// trunk body it hangs on and, where M is factored, its share of the trunk's
// rows of the factor (the Schur complement sum_D L[D][K] L[D][J] over its DoFs D,
// and the same with y), all parked in LDS as rows of 64 lanes. The trunk's
// solution goes back the same way.
#pragma once

#include "rbd_lane.hpp"
#include "rbd_team_plan.hpp"

namespace rbd {

template <class TP>
struct Team {
  static constexpr TeamPlan kPlan = team_plan(TP::kFree, TP::N, TP::par_.v);
  static constexpr bool kOn = TP::NV > kTeamMinDofs && kPlan.waves > 1;
  // the largest batch that runs OP as a team (0: none)
  template <TeamOp OP>
  static constexpr long long kLimit = kOn ? team_limit(kPlan, TP::NV, OP) : 0;
  static constexpr int kWaves = kOn ? kPlan.waves : 1;
  static constexpr int kThreads = kWaves * kTileLanes;
  static constexpr int kOwner = kPlan.owner;

  static constexpr bool trunk(int i) { return kPlan.wave[i] < 0; }
  static constexpr bool in(int w, int i) { return kPlan.wave[i] == w; }
  // trunk body a carries branches of wave w (directly or through other trunk bodies)
  static constexpr bool above(int w, int a) {
    if (!trunk(a)) return false;
    for (int i = a + 1; i <= TP::last(a); ++i)
      if (in(w, i)) return true;
    return false;
  }
  // a branch of wave w hangs on trunk body a
  static constexpr bool attach(int w, int a) {
    if (!trunk(a)) return false;
    for (int i = a + 1; i <= TP::last(a); ++i)
      if (in(w, i) && TP::parent(i) == a) return true;
    return false;
  }
  // wave w runs its own code (another wave's code with moved bodies otherwise)
  static constexpr bool own_code(int w) { return kPlan.role[w] == w; }
  // wave w or the waves that run its code include the owner
  static constexpr bool may_own(int w) { return kPlan.role[kOwner] == w; }
};

// What the waves hand to the trunk: rows of LDS (64 lanes each). For every
// trunk body a wave's branches hang on, A rows (forces and the like); for
// every trunk DoF K above them, S = true: ddepth(K) + 1 rows of the Schur
// complement (K's ancestors, then K) and R rows of right-hand sides.
// (Tables, looked up with constant indices, fold away wherever they are asked.)
template <class TP, int A, bool S, int R>
struct TeamRowTab {
  int arow[kTeamWaves][TP::N], krow[kTeamWaves][TP::NV], base[kTeamWaves + 1];
  static constexpr TeamRowTab make() {
    TeamRowTab t = {};
    for (int w = 0; w < Team<TP>::kWaves; ++w) {
      int n = 0;
      for (int a = 0; a < TP::N; ++a) {
        t.arow[w][a] = n;
        n += Team<TP>::attach(w, a) ? A : 0;
      }
      for (int k = 0; k < TP::NV; ++k) {
        t.krow[w][k] = n;
        if (Team<TP>::above(w, TP::body_of(k))) n += (S ? TP::ddepth(k) + 1 : 0) + R;
      }
      t.base[w + 1] = t.base[w] + n;
    }
    return t;
  }
};
template <class TP, int A, bool S, int R>
struct TeamRows {
  static constexpr int kRhs = R;
  static constexpr TeamRowTab<TP, A, S, R> v = TeamRowTab<TP, A, S, R>::make();
  static constexpr int arow(int w, int a) { return v.arow[w][a]; }
  // entry (k, j) of the Schur complement, j an ancestor of k or k itself
  static constexpr int srow(int w, int k, int j) { return v.krow[w][k] + TP::ddepth(j); }
  static constexpr int yrow(int w, int k, int r) { return v.krow[w][k] + (S ? TP::ddepth(k) + 1 : 0) + r; }
  static constexpr int base(int w) { return v.base[w]; }  // first row of wave w
  static constexpr int total() { return v.base[Team<TP>::kWaves]; }
};
// Rows of the trunk's DoFs, in order (the trunk's solution).
template <class TP>
struct TrunkRowTab {
  int row[TP::NV + 1];
  static constexpr TrunkRowTab make() {
    TrunkRowTab t = {};
    for (int k = 0; k < TP::NV; ++k) t.row[k + 1] = t.row[k] + (Team<TP>::trunk(TP::body_of(k)) ? 1 : 0);
    return t;
  }
};
template <class TP>
struct TrunkRows {
  static constexpr TrunkRowTab<TP> v = TrunkRowTab<TP>::make();
  static constexpr int row(int k) { return v.row[k]; }
  static constexpr int total() { return v.row[TP::NV]; }
  static constexpr int body(int i) {  // trunk bodies before body i
    int n = 0;
    for (int j = 0; j < i; ++j) n += Team<TP>::trunk(j) ? 1 : 0;
    return n;
  }
};

// Floats of a block's LDS for a number of rows. One row at least: where every
// branch hangs on the world nothing is handed over, and an array may not be empty.
constexpr int team_lds(int rows) { return (rows > 0 ? rows : 1) * kTileLanes; }

// A lane's column of a run of LDS rows.
struct LdsCol {
  float* p;
  RBD_DI void put(int row, float v) const { p[row * kTileLanes] = v; }
  RBD_DI float get(int row) const { return p[row * kTileLanes]; }
  RBD_DI LdsCol at(int row) const { return {p + row * kTileLanes}; }
};
RBD_DI void put_frc(const LdsCol& c, int row, const Frc& f) {
  c.put(row, f.n.x); c.put(row + 1, f.n.y); c.put(row + 2, f.n.z);
  c.put(row + 3, f.f.x); c.put(row + 4, f.f.y); c.put(row + 5, f.f.z);
}
RBD_DI Frc get_frc(const LdsCol& c, int row) {
  return {{c.get(row), c.get(row + 1), c.get(row + 2)}, {c.get(row + 3), c.get(row + 4), c.get(row + 5)}};
}
RBD_DI void put_inr(const LdsCol& c, int row, const Inr& I) {
  c.put(row, I.m); c.put(row + 1, I.h.x); c.put(row + 2, I.h.y); c.put(row + 3, I.h.z);
  c.put(row + 4, I.xx); c.put(row + 5, I.yy); c.put(row + 6, I.zz);
  c.put(row + 7, I.xy); c.put(row + 8, I.xz); c.put(row + 9, I.yz);
}
RBD_DI Inr get_inr(const LdsCol& c, int row) {
  return {c.get(row), {c.get(row + 1), c.get(row + 2), c.get(row + 3)}, c.get(row + 4), c.get(row + 5),
          c.get(row + 6), c.get(row + 7), c.get(row + 8), c.get(row + 9)};
}

// Where a wave finds its own branches: the wave that runs the code of role W
// with its bodies moved by `shift` reads and writes branch rows that much
// further on; trunk rows stay where they are.
struct TeamLane {
  int wave;       // uniform
  int shift;      // bodies, uniform
  uint32_t lane;  // 0..63
  uint32_t b;     // the lane's instance; lanes past the batch redo the last one
};

// The first instance of the calling block (see team_grid).
RBD_DI uint32_t team_first() { return (blockIdx.y * kTeamRowBlocks + blockIdx.x) * kTileLanes; }

// Calls body(ic<W>, TeamLane) with W the role of the calling wave, for the 64
// instances from `first` of `batch`. The branch is the same for a whole wave,
// and every wave meets the barriers inside.
template <class TP, class F>
RBD_DI void team_roles(uint32_t first, int64_t batch, F&& body) {
  using TM = Team<TP>;
  TeamLane tl;
  tl.wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kTileLanes);
  tl.lane = threadIdx.x % kTileLanes;
  const uint32_t b = first + tl.lane;
  tl.b = b < batch ? b : (uint32_t)(batch - 1);
  int role = 0;
  tl.shift = 0;
  sfor<0, TM::kWaves>([&](auto W_) __attribute__((always_inline)) {
    constexpr int W = decltype(W_)::value;
    if (tl.wave == W) {
      role = TM::kPlan.role[W];
      tl.shift = TM::kPlan.shift[W];
    }
  });
  sfor<0, TM::kWaves>([&](auto W_) __attribute__((always_inline)) {
    constexpr int W = decltype(W_)::value;
    if constexpr (TM::own_code(W)) {
      if (role == W) body(W_, tl);
    }
  });
}

// The same with every wave running its own code (its bodies in place): for
// what differs between copies of a branch, as the zeros of a matrix's rows do.
template <class TP, class F>
RBD_DI void team_waves(uint32_t first, int64_t batch, F&& body) {
  TeamLane tl;
  tl.wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kTileLanes);
  tl.shift = 0;
  tl.lane = threadIdx.x % kTileLanes;
  const uint32_t b = first + tl.lane;
  tl.b = b < batch ? b : (uint32_t)(batch - 1);
  sfor<0, Team<TP>::kWaves>([&](auto W_) __attribute__((always_inline)) {
    constexpr int W = decltype(W_)::value;
    if (tl.wave == W) body(W_, tl);
  });
}

// The row base of the calling wave among those that run the code of role W.
template <class TP, class ROWS, int W>
RBD_DI int team_base(const TeamLane& tl) {
  using TM = Team<TP>;
  int base = ROWS::base(W);
  sfor<W + 1, TM::kWaves>([&](auto V_) __attribute__((always_inline)) {
    constexpr int V = decltype(V_)::value;
    if constexpr (TM::kPlan.role[V] == W) {
      if (tl.wave == V) base = cidx<ROWS::base(V)>;
    }
  });
  return base;
}

// Loads what role W reads of an input vector: entries of its own branches from
// the moved view `br`, of the trunk bodies above them (ABOVE) from `tk`.
// DOF: one entry per DoF (6 for a free base), else the entries of q.
template <class TP, int W, bool ABOVE, bool DOF, class V, int n>
RBD_DI void team_load(float (&x)[n], const V& br, const V& tk) {
  using TM = Team<TP>;
  sfor<0, TP::N>([&](auto I_) __attribute__((always_inline)) {
    constexpr int I = decltype(I_)::value;
    constexpr int o = DOF ? TP::vofs(I) : TP::qofs(I);
    if constexpr (TM::in(W, I)) {
      x[o] = br(o);
    } else if constexpr (ABOVE && TM::above(W, I)) {
      sfor<0, (TP::free_body(I) ? (DOF ? 6 : 7) : 1)>([&](auto C_) __attribute__((always_inline)) {
        x[o + decltype(C_)::value] = tk(o + decltype(C_)::value);
      });
    }
  });
}

// The same for all of the trunk (what the owner reads).
template <class TP, bool DOF, class V, int n>
RBD_DI void team_load_trunk(float (&x)[n], const V& tk) {
  sfor<0, TP::N>([&](auto I_) __attribute__((always_inline)) {
    constexpr int I = decltype(I_)::value;
    constexpr int o = DOF ? TP::vofs(I) : TP::qofs(I);
    if constexpr (Team<TP>::trunk(I)) {
      sfor<0, (TP::free_body(I) ? (DOF ? 6 : 7) : 1)>([&](auto C_) __attribute__((always_inline)) {
        x[o + decltype(C_)::value] = tk(o + decltype(C_)::value);
      });
    }
  });
}

// f(column of rows) for every wave that left rows for trunk body J, in order.
template <class TP, class ROWS, int J, class F>
RBD_DI void team_collect(const LdsCol& lds, const F& f) {
  sfor<0, Team<TP>::kWaves>([&](auto W_) __attribute__((always_inline)) {
    constexpr int W = decltype(W_)::value;
    if constexpr (Team<TP>::attach(W, J)) f(lds.at(cidx<ROWS::base(W) + ROWS::arow(W, J)>));
  });
}

// =================================================================== forward dynamics
// The state of the bias and mass-matrix sweep (see fwd_dyn_lane); only the
// entries of the bodies a wave visits are ever used.
template <class TP, bool EXT>
struct TeamFd {
  M3 R[TP::N];
  Mot v[TP::N], a[TP::N];
  Frc f[TP::N];
  Inr Ic[TP::N];
  M3 Rw[EXT ? TP::N : 1];
  V3 pw[EXT ? TP::N : 1];
};

// Motion and force of body I (see body_motion), and its world pose where there
// are external forces.
template <class TP, int I, bool QDD = false, class QI, class QDI, class ST, class FX>
RBD_DI void team_fd_motion(const float* __restrict__ t, const QI& q, const QDI& qd, V3 mg, ST& s, const FX&) {
  body_motion<TP, I, QDD>(t, q, qd, mg, s.R, s.v, s.a);
  if constexpr (FX::kOn) world_pose<TP, I>(t, q, s.R[I], s.Rw, s.pw);
}
template <class TP, int I, bool QDD = false, class ST, class FX>
RBD_DI void team_fd_force(const float* __restrict__ t, ST& s, const FX& fx) {
  s.f[I] = body_force<TP, I, QDD>(t, s.v, s.a);
  if constexpr (FX::kOn) s.f[I] = s.f[I] - fext_body<I>(fx, s.Rw[I], s.pw[I]);
}

// The trunk's rows of the factor only see the trunk's own rows: the branches'
// share has been taken off the mass matrix already.
template <class TP>
struct TrunkDofs {
  static constexpr bool on(int k) { return Team<TP>::trunk(TP::body_of(k)); }
};

// walk_up over a branch of a wave and on over the trunk.
template <class TP, int C, class EMIT>
RBD_DI void team_walk_up(const float* __restrict__ t, const float* __restrict__ tb, const M3* R, Frc F, EMIT& emit) {
  constexpr int A = TP::parent(C);
  if constexpr (A >= 0) {
    F = xfrc(R[C], load_r<C>(Team<TP>::trunk(C) ? t : tb), F);
    emit(ic<A>{}, F);
    team_walk_up<TP, A>(t, tb, R, F, emit);
  }
}

// Branch W's share of trunk DoF K's right-hand side r.
template <class TP, int W, int K, int r, class MASK = AllRhs, int NRHS>
RBD_DI float team_yshare(const Ltl<TP, NRHS>& F) {
  float acc = 0.0f;
  sfor<K + 1, cidx<TP::dlast(K)> + 1>([&](auto D_) __attribute__((always_inline)) {
    constexpr int D = decltype(D_)::value;
    if constexpr (Team<TP>::in(W, TP::body_of(D)) && MASK::on(r, D))
      acc = __builtin_fmaf(F.L[cidx<TP::lidx(D, K)>], F.y[r][D], acc);
  });
  return acc;
}

// What a caller adds to the sweep up: after a body's motion, its right-hand
// sides (the bias force is taken off the first by default), after its row of
// the factor.
template <class RHS>
struct FdHook {
  const RHS& rhs;
  template <class I, class ST>
  RBD_DI void motion(I, const ST&) const {}
  template <class J, class ST, int n>
  RBD_DI void sides(J, int k, const ST& s, float (&b)[n]) const {
#pragma unroll
    for (int r = 0; r < n; ++r) b[r] = r == 0 ? rhs(r, k) - s.f[J::value].n.z : rhs(r, k);
  }
  template <class ST, int n>
  RBD_DI void base_sides(int k, const ST& s, float (&b)[n]) const {
    const float hb[6] = {s.f[0].f.x, s.f[0].f.y, s.f[0].f.z, s.f[0].n.x, s.f[0].n.y, s.f[0].n.z};
#pragma unroll
    for (int r = 0; r < n; ++r) b[r] = rhs(r, k) - (r == 0 ? hb[k] : 0.0f);
  }
  template <class J, class ST, class LF>
  RBD_DI void closed(J, const ST&, const LF&) const {}
};

// Role W, up: its branches' rows of the factor, from the leaves to the trunk,
// and their share of the trunk's (to LDS at `c`; of the right-hand sides the
// ROWS::kRhs first).
template <class TP, int W, int NRHS, class ROWS, class MASK = AllRhs, class QV, class QDV, class HOOK, class FX,
          class ST>
RBD_DI void team_fd_up(const float* __restrict__ t, const float* __restrict__ tb, const QV& q, const QDV& qd,
                       HOOK&& hook, const FX& fx, ST& s, Ltl<TP, NRHS>& F, const LdsCol& c) {
  using TM = Team<TP>;
  constexpr int N = TP::N, NV = TP::NV;
  const V3 g = load_g<TP>(t);
  const V3 mg = {-g.x, -g.y, -g.z};
  auto backward = [&](auto J_) __attribute__((always_inline)) {
    constexpr int J = decltype(J_)::value;
    constexpr int P = TP::parent(J);
    if constexpr (TM::in(W, J)) {
      constexpr int k = TP::vofs(J);
      // own inertias are read again where they enter (see fwd_dyn_lane)
      const float* const tc = opaque_table(tb);
      if constexpr (TP::last(J) == J) s.Ic[J] = load_inr<J>(tc);
      float Mr[NV];
      {
        auto emit = [&](auto A_, const Frc& e) __attribute__((always_inline)) {
          constexpr int A = decltype(A_)::value;
          if constexpr (TP::free_body(A)) {
            Mr[0] = e.f.x; Mr[1] = e.f.y; Mr[2] = e.f.z;
            Mr[3] = e.n.x; Mr[4] = e.n.y; Mr[5] = e.n.z;
          } else {
            Mr[cidx<TP::vofs(A)>] = e.n.z;
          }
        };
        team_walk_up<TP, J>(t, tb, s.R, inr_col_z(s.Ic[J]), emit);
      }
      float bk[NRHS];
      hook.sides(J_, k, s, bk);
      ltl_row<TP, k, NRHS, MASK>(F, Mr, s.Ic[J].zz, bk);
      hook.closed(J_, s, F);
      if constexpr (P >= 0) {
        const V3 r = load_r<J>(tb);
        xfrc_acc(s.R[J], r, s.f[J], s.f[P]);
        if constexpr (J == P + 1 && TM::in(W, P)) s.Ic[P] = load_inr<P>(tc);
        xinr_acc(s.R[J], r, s.Ic[J], s.Ic[P]);
      }
    }
  };
  sfor<0, N>([&](auto I_) __attribute__((always_inline)) {
    constexpr int I = decltype(I_)::value;
    if constexpr (TM::above(W, I)) {
      team_fd_motion<TP, I>(t, q, qd, mg, s, fx);
      hook.motion(I_, s);
      if constexpr (TM::attach(W, I)) {  // sums what the branches exert on it
        s.f[I] = Frc{};
        s.Ic[I] = Inr{};
      }
    } else if constexpr (TM::in(W, I)) {
      team_fd_motion<TP, I>(tb, q, qd, mg, s, fx);
      hook.motion(I_, s);
      team_fd_force<TP, I>(tb, s, fx);
      close_subtrees<TP, I, I>(backward);
    }
  });
  // to the trunk
  sfor<0, N>([&](auto I_) __attribute__((always_inline)) {
    constexpr int I = decltype(I_)::value;
    if constexpr (TM::attach(W, I)) {
      put_frc(c, ROWS::arow(W, I), s.f[I]);
      put_inr(c, ROWS::arow(W, I) + 6, s.Ic[I]);
    }
  });
  sfor<0, NV>([&](auto K_) __attribute__((always_inline)) {
    constexpr int K = decltype(K_)::value;
    if constexpr (TM::above(W, TP::body_of(K))) {
      sfor<0, K + 1>([&](auto J_) __attribute__((always_inline)) {
        constexpr int J = decltype(J_)::value;
        if constexpr (J == K || TP::is_danc(J, K)) {
          float acc = 0.0f;
          sfor<K + 1, cidx<TP::dlast(K)> + 1>([&](auto D_) __attribute__((always_inline)) {
            constexpr int D = decltype(D_)::value;
            if constexpr (TM::in(W, TP::body_of(D)))
              acc = __builtin_fmaf(F.L[cidx<TP::lidx(D, K)>], F.L[cidx<TP::lidx(D, J)>], acc);
          });
          c.put(cidx<ROWS::srow(W, K, J)>, acc);
        }
      });
      sfor<0, ROWS::kRhs>([&](auto R_) __attribute__((always_inline)) {
        constexpr int r = decltype(R_)::value;
        c.put(cidx<ROWS::yrow(W, K, r)>, team_yshare<TP, W, K, r>(F));
      });
    }
  });
}

// The owner's half of the way down: motion and force of the trunk
// bodies (those above its own branches have their motion already).
template <class TP, int W, class QV, class QDV, class FX, class ST>
RBD_DI void team_fd_trunk_down(const float* __restrict__ t, const QV& q, const QDV& qd, const FX& fx, ST& s) {
  using TM = Team<TP>;
  const V3 g = load_g<TP>(t);
  const V3 mg = {-g.x, -g.y, -g.z};
  sfor<0, TP::N>([&](auto I_) __attribute__((always_inline)) {
    constexpr int I = decltype(I_)::value;
    if constexpr (TM::trunk(I)) {
      if constexpr (!TM::above(W, I)) team_fd_motion<TP, I>(t, q, qd, mg, s, fx);
      team_fd_force<TP, I>(t, s, fx);
    }
  });
}

// The trunk, leaves to root: takes over what the branches left in LDS and
// factors the trunk's rows.
template <class TP, int NRHS, class ROWS, class MASK = AllRhs, class ST, class HOOK>
RBD_DI void team_fd_trunk(const float* __restrict__ t, HOOK&& hook, ST& s, const LdsCol& lds, Ltl<TP, NRHS>& F) {
  using TM = Team<TP>;
  constexpr int N = TP::N, NV = TP::NV;
  // row K of the factor: the mass matrix less what the branches have used up
  auto row = [&](auto K_, float* Mr, float Mkk, float* bk) __attribute__((always_inline)) {
    constexpr int K = decltype(K_)::value;
    sfor<0, TM::kWaves>([&](auto W_) __attribute__((always_inline)) {
      constexpr int W = decltype(W_)::value;
      if constexpr (TM::above(W, TP::body_of(K))) {
        const LdsCol c = lds.at(cidx<ROWS::base(W)>);
        sfor<0, K>([&](auto J_) __attribute__((always_inline)) {
          constexpr int J = decltype(J_)::value;
          if constexpr (TP::is_danc(J, K)) Mr[J] = Mr[J] - c.get(cidx<ROWS::srow(W, K, J)>);
        });
        Mkk = Mkk - c.get(cidx<ROWS::srow(W, K, K)>);
#pragma unroll
        for (int r = 0; r < ROWS::kRhs; ++r) bk[r] = bk[r] - c.get(cidx<ROWS::yrow(W, K, 0)> + r);
      }
    });
    ltl_row<TP, K, NRHS, MASK, TrunkDofs<TP>>(F, Mr, Mkk, bk);
  };
  sfor<0, N>([&](auto I_) __attribute__((always_inline)) {
    constexpr int I = decltype(I_)::value;
    if constexpr (TM::trunk(I)) s.Ic[I] = load_inr<I>(t);
  });
  sfor_rev<0, N>([&](auto J_) __attribute__((always_inline)) {
    constexpr int J = decltype(J_)::value;
    constexpr int P = TP::parent(J);
    if constexpr (TM::trunk(J)) {
      team_collect<TP, ROWS, J>(lds, [&](const LdsCol& c) __attribute__((always_inline)) {
        s.f[J] = s.f[J] + get_frc(c, 0);
        s.Ic[J] = s.Ic[J] + get_inr(c, 6);
      });
      if constexpr (TP::free_body(J)) {
        sfor_rev<0, 6>([&](auto K_) __attribute__((always_inline)) {
          constexpr int K = decltype(K_)::value;
          float Mr[6], bk[NRHS];
#pragma unroll
          for (int j = 0; j < K; ++j) Mr[j] = base_block(s.Ic[J], K, j);
          hook.base_sides(K, s, bk);
          row(K_, Mr, base_block(s.Ic[J], K, K), bk);
        });
        hook.closed(J_, s, F);
      } else {
        constexpr int k = TP::vofs(J);
        float Mr[NV], bk[NRHS];
        crba_row<TP, J>(t, s.R, s.Ic[J], Mr);
        hook.sides(J_, k, s, bk);
        row(ic<k>{}, Mr, s.Ic[J].zz, bk);
        hook.closed(J_, s, F);
        if constexpr (P >= 0) {
          const V3 r = load_r<J>(t);
          xfrc_acc(s.R[J], r, s.f[J], s.f[P]);
          xinr_acc(s.R[J], r, s.Ic[J], s.Ic[P]);
        }
      }
    }
  });
}

// Role W, down: x of its branches, given the trunk's (xt(r, k)).
template <class TP, int W, int NRHS, class XT, class SINK>
RBD_DI void team_fd_back(const Ltl<TP, NRHS>& F, const XT& xt, const SINK& sink) {
  using TM = Team<TP>;
  constexpr int NV = TP::NV;
  sfor<0, NRHS>([&](auto R_) __attribute__((always_inline)) {
    constexpr int r = decltype(R_)::value;
    float x[NV];
    sfor<0, NV>([&](auto K_) __attribute__((always_inline)) {
      constexpr int K = decltype(K_)::value;
      if constexpr (TM::above(W, TP::body_of(K))) {
        x[K] = xt(r, K);
      } else if constexpr (TM::in(W, TP::body_of(K))) {
        float acc = F.y[r][K];
        sfor<0, K>([&](auto J_) __attribute__((always_inline)) {
          constexpr int Jd = decltype(J_)::value;
          if constexpr (TP::is_danc(Jd, K)) acc = acc - F.L[cidx<TP::lidx(K, Jd)>] * x[Jd];
        });
        x[K] = acc * F.Linv[K];
        sink(r, K, x[K]);
      }
    });
  });
}

// Forward dynamics of role W with NRHS right-hand sides, three phases with a
// barrier between: the branches up (rhs reads branch entries), the trunk by the
// owner (rhs_t reads trunk entries), the branches down. q, qd: the role's and,
// for the owner, the trunk's entries. xrow keeps the trunk's solution, one run
// of rows per right-hand side; F the role's rows of the factor, Ft the trunk's
// (owner). sink(r, k, x) gets the role's branches, sink_t the trunk (owner).
template <class TP, int W, int NRHS, class ROWS, class QV, class QDV, class RHS, class RHST, class FX, class SINK,
          class SINKT>
RBD_DI void team_fd(const TeamLane& tl, bool owner, const float* __restrict__ tab, const QV& q, const QDV& qd,
                    const RHS& rhs, const RHST& rhs_t, const FX& fxb, const FX& fx, const LdsCol& lds,
                    const LdsCol& xrow, Ltl<TP, NRHS>& F, Ltl<TP, NRHS>& Ft, const SINK& sink, const SINKT& sink_t) {
  using TM = Team<TP>;
  constexpr int T = TrunkRows<TP>::total();
  TeamFd<TP, FX::kOn> s;
  const float* const t = opaque_table(tab);
  team_fd_up<TP, W, NRHS, ROWS>(t, opaque_table(tab + tl.shift * kBodyStride), q, qd, FdHook<RHS>{rhs}, fxb, s, F,
                                lds.at(team_base<TP, ROWS, W>(tl)));
  if constexpr (TM::may_own(W)) {
    if (owner) team_fd_trunk_down<TP, W>(t, q, qd, fx, s);
  }
  __syncthreads();
  if constexpr (TM::may_own(W)) {
    if (owner) {
      team_fd_trunk<TP, NRHS, ROWS>(t, FdHook<RHST>{rhs_t}, s, lds, Ft);
      ltl_back<TP, NRHS, TrunkDofs<TP>>(Ft, [&](int r, int k, float x) __attribute__((always_inline)) {
        xrow.put(r * T + TrunkRows<TP>::row(k), x);
        sink_t(r, k, x);
      });
    }
  }
  __syncthreads();
  team_fd_back<TP, W, NRHS>(
      F, [&](int r, int k) __attribute__((always_inline)) { return xrow.get(r * T + TrunkRows<TP>::row(k)); }, sink);
}

// =================================================================== inverse dynamics
// Role W: torques of its branches; the force on the trunk goes to LDS.
template <class TP, int W, class ROWS, bool HAS_QDD, class QV, class QDV, class QDDV, class FX, class ST, class TO>
RBD_DI void team_id_up(const float* __restrict__ t, const float* __restrict__ tb, const QV& q, const QDV& qd,
                       const QDDV& qdd, const FX& fx, ST& s, const LdsCol& c, const TO& tau) {
  using TM = Team<TP>;
  const V3 g = load_g<TP>(t);
  const V3 mg = {-g.x, -g.y, -g.z};
  auto backward = [&](auto J_) __attribute__((always_inline)) {
    constexpr int J = decltype(J_)::value;
    constexpr int P = TP::parent(J);
    if constexpr (TM::in(W, J)) {
      tau(cidx<TP::vofs(J)>, s.f[J].n.z);
      if constexpr (P >= 0) xfrc_acc(s.R[J], load_r<J>(tb), s.f[J], s.f[P]);
    }
  };
  sfor<0, TP::N>([&](auto I_) __attribute__((always_inline)) {
    constexpr int I = decltype(I_)::value;
    if constexpr (TM::above(W, I)) {
      team_fd_motion<TP, I, HAS_QDD>(t, q, qd, mg, s, fx);
      if constexpr (HAS_QDD) add_qdd<TP, I>(s.a, qdd);
      if constexpr (TM::attach(W, I)) s.f[I] = Frc{};
    } else if constexpr (TM::in(W, I)) {
      team_fd_motion<TP, I, HAS_QDD>(tb, q, qd, mg, s, fx);
      if constexpr (HAS_QDD) add_qdd<TP, I>(s.a, qdd);
      team_fd_force<TP, I, HAS_QDD>(tb, s, fx);
      close_subtrees<TP, I, I>(backward);
    }
  });
  sfor<0, TP::N>([&](auto I_) __attribute__((always_inline)) {
    constexpr int I = decltype(I_)::value;
    if constexpr (TM::attach(W, I)) put_frc(c, ROWS::arow(W, I), s.f[I]);
  });
}
template <class TP, int W, bool HAS_QDD, class QV, class QDV, class QDDV, class FX, class ST>
RBD_DI void team_id_trunk_down(const float* __restrict__ t, const QV& q, const QDV& qd, const QDDV& qdd, const FX& fx,
                               ST& s) {
  using TM = Team<TP>;
  const V3 g = load_g<TP>(t);
  const V3 mg = {-g.x, -g.y, -g.z};
  sfor<0, TP::N>([&](auto I_) __attribute__((always_inline)) {
    constexpr int I = decltype(I_)::value;
    if constexpr (TM::trunk(I)) {
      if constexpr (!TM::above(W, I)) {
        team_fd_motion<TP, I, HAS_QDD>(t, q, qd, mg, s, fx);
        if constexpr (HAS_QDD) add_qdd<TP, I>(s.a, qdd);
      }
      team_fd_force<TP, I, HAS_QDD>(t, s, fx);
    }
  });
}
template <class TP, class ROWS, class ST, class TO>
RBD_DI void team_id_trunk(const float* __restrict__ t, ST& s, const LdsCol& lds, const TO& tau) {
  using TM = Team<TP>;
  sfor_rev<0, TP::N>([&](auto J_) __attribute__((always_inline)) {
    constexpr int J = decltype(J_)::value;
    constexpr int P = TP::parent(J);
    if constexpr (TM::trunk(J)) {
      team_collect<TP, ROWS, J>(
          lds, [&](const LdsCol& c) __attribute__((always_inline)) { s.f[J] = s.f[J] + get_frc(c, 0); });
      if constexpr (TP::free_body(J)) {
        tau(0, s.f[J].f.x); tau(1, s.f[J].f.y); tau(2, s.f[J].f.z);
        tau(3, s.f[J].n.x); tau(4, s.f[J].n.y); tau(5, s.f[J].n.z);
      } else {
        tau(cidx<TP::vofs(J)>, s.f[J].n.z);
        if constexpr (P >= 0) xfrc_acc(s.R[J], load_r<J>(t), s.f[J], s.f[P]);
      }
    }
  });
}

// =================================================================== adjoint of inverse dynamics
// Role W: the outputs of its branches (see id_adjoint_lane); its share of the
// trunk's totals goes to LDS.
template <class TP, int W, class ROWS, class ST, class QV, class QDV, class QDDV, class LAM, class GQ, class GQD,
          class FX, class GF, class GQDD>
RBD_DI void team_adj_up(const float* __restrict__ t, const float* __restrict__ tb, ST& s, const QV& q, const QDV& qd,
                        const QDDV& qdd, const LAM& lam, const GQ& gq, const GQD& gqd, const FX& fx, const GF& gf,
                        const GQDD& gqdd, const LdsCol& c) {
  using TM = Team<TP>;
  const V3 g = load_g<TP>(t);
  const V3 mg = {-g.x, -g.y, -g.z};
  auto backward = [&](auto J_) __attribute__((always_inline)) {
    constexpr int J = decltype(J_)::value;
    if constexpr (TM::in(W, J)) adj_close<TP, J>(tb, g, s, q, qd, gq, gqd, gqdd);
  };
  sfor<0, TP::N>([&](auto I_) __attribute__((always_inline)) {
    constexpr int I = decltype(I_)::value;
    if constexpr (TM::above(W, I)) {
      adj_motion<TP, I>(t, mg, s, q, qd, qdd, lam);
      if constexpr (TM::attach(W, I)) {  // sums what the branches add to its totals
        s.f[I] = Frc{};
        s.ab[I] = Frc{};
        s.vb[I] = Frc{};
        if constexpr (ST::kExt) {
          s.Fs[I] = Frc{};
          s.Ws[I] = Frc{};
        }
      }
    } else if constexpr (TM::in(W, I)) {
      adj_motion<TP, I>(tb, mg, s, q, qd, qdd, lam);
      adj_force<TP, I>(tb, s, fx, gf);
      close_subtrees<TP, I, I>(backward);
    }
  });
  sfor<0, TP::N>([&](auto I_) __attribute__((always_inline)) {
    constexpr int I = decltype(I_)::value;
    if constexpr (TM::attach(W, I)) {
      constexpr int r = ROWS::arow(W, I);
      put_frc(c, r, s.f[I]);
      put_frc(c, r + 6, s.ab[I]);
      put_frc(c, r + 12, s.vb[I]);
      if constexpr (ST::kExt) {
        put_frc(c, r + 18, s.Fs[I]);
        put_frc(c, r + 24, s.Ws[I]);
      }
    }
  });
}
template <class TP, int W, class ST, class QV, class QDV, class QDDV, class LAM, class FX, class GF>
RBD_DI void team_adj_trunk_down(const float* __restrict__ t, ST& s, const QV& q, const QDV& qd, const QDDV& qdd,
                                const LAM& lam, const FX& fx, const GF& gf) {
  using TM = Team<TP>;
  const V3 g = load_g<TP>(t);
  const V3 mg = {-g.x, -g.y, -g.z};
  sfor<0, TP::N>([&](auto I_) __attribute__((always_inline)) {
    constexpr int I = decltype(I_)::value;
    if constexpr (TM::trunk(I)) {
      if constexpr (!TM::above(W, I)) adj_motion<TP, I>(t, mg, s, q, qd, qdd, lam);
      adj_force<TP, I>(t, s, fx, gf);
    }
  });
}
template <class TP, class ROWS, class ST, class QV, class QDV, class GQ, class GQD, class GQDD>
RBD_DI void team_adj_trunk(const float* __restrict__ t, ST& s, const QV& q, const QDV& qd, const GQ& gq,
                           const GQD& gqd, const GQDD& gqdd, const LdsCol& lds) {
  const V3 g = load_g<TP>(t);
  sfor_rev<0, TP::N>([&](auto J_) __attribute__((always_inline)) {
    constexpr int J = decltype(J_)::value;
    if constexpr (Team<TP>::trunk(J)) {
      team_collect<TP, ROWS, J>(lds, [&](const LdsCol& c) __attribute__((always_inline)) {
        s.f[J] = s.f[J] + get_frc(c, 0);
        s.ab[J] = s.ab[J] + get_frc(c, 6);
        s.vb[J] = s.vb[J] + get_frc(c, 12);
        if constexpr (ST::kExt) {
          s.Fs[J] = s.Fs[J] + get_frc(c, 18);
          s.Ws[J] = s.Ws[J] + get_frc(c, 24);
        }
      });
      adj_close<TP, J>(t, g, s, q, qd, gq, gqd, gqdd);
    }
  });
}

// =================================================================== tangent of inverse dynamics
// Role W: the outputs of its branches (see id_tangent_lane); the forces on
// the trunk and their tangents go to LDS.
template <class TP, int W, class ROWS, class ST, class QV, class QDV, class QDDV, class DQV, class DQDV, class DQDDV,
          class DT, class FX, class DFX, class OUT>
RBD_DI void team_tan_up(const float* __restrict__ t, const float* __restrict__ tb, ST& s, const QV& q, const QDV& qd,
                        const QDDV& qdd, const DQV& dq, const DQDV& dqd, const DQDDV& dqdd, const DT& dtau,
                        const FX& fx, const DFX& dfx, const LdsCol& c, const OUT& out) {
  using TM = Team<TP>;
  const V3 g = load_g<TP>(t);
  const V3 mg = {-g.x, -g.y, -g.z};
  auto backward = [&](auto J_) __attribute__((always_inline)) {
    constexpr int J = decltype(J_)::value;
    if constexpr (TM::in(W, J)) tan_close<TP, J>(tb, s, dq, dtau, out);
  };
  sfor<0, TP::N>([&](auto I_) __attribute__((always_inline)) {
    constexpr int I = decltype(I_)::value;
    if constexpr (TM::above(W, I)) {
      tan_motion<TP, I>(t, mg, s, q, qd, qdd, dq, dqd, dqdd);
      if constexpr (TM::attach(W, I)) {
        s.f[I] = Frc{};
        s.df[I] = Frc{};
      }
    } else if constexpr (TM::in(W, I)) {
      tan_motion<TP, I>(tb, mg, s, q, qd, qdd, dq, dqd, dqdd);
      tan_force<TP, I>(tb, s, fx, dfx);
      close_subtrees<TP, I, I>(backward);
    }
  });
  sfor<0, TP::N>([&](auto I_) __attribute__((always_inline)) {
    constexpr int I = decltype(I_)::value;
    if constexpr (TM::attach(W, I)) {
      put_frc(c, ROWS::arow(W, I), s.f[I]);
      put_frc(c, ROWS::arow(W, I) + 6, s.df[I]);
    }
  });
}
template <class TP, int W, class ST, class QV, class QDV, class QDDV, class DQV, class DQDV, class DQDDV, class FX,
          class DFX>
RBD_DI void team_tan_trunk_down(const float* __restrict__ t, ST& s, const QV& q, const QDV& qd, const QDDV& qdd,
                                const DQV& dq, const DQDV& dqd, const DQDDV& dqdd, const FX& fx, const DFX& dfx) {
  using TM = Team<TP>;
  const V3 g = load_g<TP>(t);
  const V3 mg = {-g.x, -g.y, -g.z};
  sfor<0, TP::N>([&](auto I_) __attribute__((always_inline)) {
    constexpr int I = decltype(I_)::value;
    if constexpr (TM::trunk(I)) {
      if constexpr (!TM::above(W, I)) tan_motion<TP, I>(t, mg, s, q, qd, qdd, dq, dqd, dqdd);
      tan_force<TP, I>(t, s, fx, dfx);
    }
  });
}
template <class TP, class ROWS, class ST, class DQV, class DT, class OUT>
RBD_DI void team_tan_trunk(const float* __restrict__ t, ST& s, const DQV& dq, const DT& dtau, const LdsCol& lds,
                           const OUT& out) {
  sfor_rev<0, TP::N>([&](auto J_) __attribute__((always_inline)) {
    constexpr int J = decltype(J_)::value;
    if constexpr (Team<TP>::trunk(J)) {
      team_collect<TP, ROWS, J>(lds, [&](const LdsCol& c) __attribute__((always_inline)) {
        s.f[J] = s.f[J] + get_frc(c, 0);
        s.df[J] = s.df[J] + get_frc(c, 6);
      });
      tan_close<TP, J>(t, s, dq, dtau, out);
    }
  });
}

// y of L^T y = b over role W's branches for a factor that is there already,
// and its share of the trunk's right-hand side (to LDS).
template <class TP, int W, class ROWS, class B>
RBD_DI void team_solve_y(Ltl<TP, 1>& F, const B& b, const LdsCol& c) {
  using TM = Team<TP>;
  sfor_rev<0, TP::NV>([&](auto K_) __attribute__((always_inline)) {
    constexpr int K = decltype(K_)::value;
    constexpr bool kOwn = TM::in(W, TP::body_of(K));
    if constexpr (kOwn || TM::above(W, TP::body_of(K))) {
      float acc = kOwn ? b(K) : 0.0f;
      sfor<K + 1, cidx<TP::dlast(K)> + 1>([&](auto D_) __attribute__((always_inline)) {
        constexpr int D = decltype(D_)::value;
        if constexpr (TM::in(W, TP::body_of(D)))
          acc = __builtin_fmaf(kOwn ? -F.L[cidx<TP::lidx(D, K)>] : F.L[cidx<TP::lidx(D, K)>], F.y[0][D], acc);
      });
      if constexpr (kOwn) F.y[0][K] = acc * F.Linv[K];
      else c.put(cidx<ROWS::yrow(W, K, 0)>, acc);
    }
  });
}
// The trunk's y, then x.
template <class TP, class ROWS, class B, class SINK>
RBD_DI void team_solve_trunk(Ltl<TP, 1>& F, const B& b, const LdsCol& lds, const SINK& sink) {
  using TM = Team<TP>;
  sfor_rev<0, TP::NV>([&](auto K_) __attribute__((always_inline)) {
    constexpr int K = decltype(K_)::value;
    if constexpr (TM::trunk(TP::body_of(K))) {
      float acc = b(K);
      sfor<0, TM::kWaves>([&](auto W_) __attribute__((always_inline)) {
        constexpr int W = decltype(W_)::value;
        if constexpr (TM::above(W, TP::body_of(K))) acc = acc - lds.get(cidx<ROWS::base(W) + ROWS::yrow(W, K, 0)>);
      });
      sfor<K + 1, cidx<TP::dlast(K)> + 1>([&](auto D_) __attribute__((always_inline)) {
        constexpr int D = decltype(D_)::value;
        if constexpr (TM::trunk(TP::body_of(D))) acc = acc - F.L[cidx<TP::lidx(D, K)>] * F.y[0][D];
      });
      F.y[0][K] = acc * F.Linv[K];
    }
  });
  ltl_back<TP, 1, TrunkDofs<TP>>(F, sink);
}

// =================================================================== articulated-body algorithm
RBD_DI void put_ainr(const LdsCol& c, int row, const AInr& I) {
  const float x[12] = {I.a00, I.a11, I.a22, I.a01, I.a02, I.a12, I.c00, I.c11, I.c22, I.c01, I.c02, I.c12};
#pragma unroll
  for (int e = 0; e < 12; ++e) c.put(row + e, x[e]);
#pragma unroll
  for (int e = 0; e < 9; ++e) c.put(row + 12 + e, I.b[e]);
}
RBD_DI void add_ainr(const LdsCol& c, int row, AInr& I) {
  float* const x[12] = {&I.a00, &I.a11, &I.a22, &I.a01, &I.a02, &I.a12, &I.c00, &I.c11, &I.c22, &I.c01, &I.c02, &I.c12};
#pragma unroll
  for (int e = 0; e < 12; ++e) *x[e] = *x[e] + c.get(row + e);
#pragma unroll
  for (int e = 0; e < 9; ++e) I.b[e] = I.b[e] + c.get(row + 12 + e);
}

// Role W, up (see aba_lane): the articulated inertia and bias force that its
// branches add to the trunk bodies they hang on go to LDS (27 rows a body).
template <class TP, int W, class ROWS, class ST, class QV, class QDV, class TV, class FX>
RBD_DI void team_aba_up(const float* __restrict__ t, const float* __restrict__ tb, ST& s, const QV& q, const QDV& qd,
                        const TV& tau, const FX& fx, const LdsCol& c) {
  using TM = Team<TP>;
  auto close = [&](auto J_) __attribute__((always_inline)) {
    constexpr int J = decltype(J_)::value;
    constexpr int P = TP::parent(J);
    if constexpr (TM::in(W, J)) {
      constexpr bool kFirst = J == P + 1 && P >= 0 && !TM::trunk(P < 0 ? 0 : P);
      aba_close<TP, J, kFirst, FX>(tb, s, qd, tau);
    }
  };
  sfor<0, TP::N>([&](auto I_) __attribute__((always_inline)) {
    constexpr int I = decltype(I_)::value;
    if constexpr (TM::above(W, I)) {
      aba_motion<TP, I>(t, s, q, qd, fx);
      if constexpr (TM::attach(W, I)) {
        s.acc[I] = AInr{};
        s.accp[I] = Frc{};
      }
    } else if constexpr (TM::in(W, I)) {
      aba_motion<TP, I>(tb, s, q, qd, fx);
      close_subtrees<TP, I, I>(close);
    }
  });
  sfor<0, TP::N>([&](auto I_) __attribute__((always_inline)) {
    constexpr int I = decltype(I_)::value;
    if constexpr (TM::attach(W, I)) {
      put_ainr(c, ROWS::arow(W, I), s.acc[I]);
      put_frc(c, ROWS::arow(W, I) + 21, s.accp[I]);
    }
  });
}
// The trunk, up and down; `acc` takes the accelerations that the branches start
// from, 6 rows per trunk body.
template <class TP, class ROWS, class FX, class ST, class QV, class QDV, class TV, class OUT>
RBD_DI void team_aba_trunk(const float* __restrict__ t, ST& s, const QV& q, const QDV& qd, const TV& tau,
                           const LdsCol& lds, const LdsCol& acc, const OUT& qdd) {
  using TM = Team<TP>;
  const V3 g = load_g<TP>(t);
  const V3 mg = {-g.x, -g.y, -g.z};
  sfor<0, TP::N>([&](auto I_) __attribute__((always_inline)) {
    constexpr int I = decltype(I_)::value;
    if constexpr (TM::trunk(I)) {
      s.acc[I] = AInr{};
      s.accp[I] = Frc{};
    }
  });
  sfor_rev<0, TP::N>([&](auto J_) __attribute__((always_inline)) {
    constexpr int J = decltype(J_)::value;
    if constexpr (TM::trunk(J)) {
      team_collect<TP, ROWS, J>(lds, [&](const LdsCol& c) __attribute__((always_inline)) {
        add_ainr(c, 0, s.acc[J]);
        s.accp[J] = s.accp[J] + get_frc(c, 21);
      });
      aba_close<TP, J, false, FX>(t, s, qd, tau);
    }
  });
  AbaDown<TP> d;
  sfor<0, TP::N>([&](auto I_) __attribute__((always_inline)) {
    constexpr int I = decltype(I_)::value;
    if constexpr (TM::trunk(I)) {
      aba_down<TP, I>(t, mg, s, d, q, qd, qdd);
      const Frc a = {d.a[I].w, d.a[I].v};
      put_frc(acc, 6 * cidx<TrunkRows<TP>::body(I)>, a);
    }
  });
}
// Role W, down.
template <class TP, int W, class ST, class QV, class QDV, class OUT>
RBD_DI void team_aba_down(const float* __restrict__ t, const float* __restrict__ tb, const ST& s, const QV& q,
                          const QDV& qd, const LdsCol& acc, const OUT& qdd) {
  using TM = Team<TP>;
  const V3 g = load_g<TP>(t);
  const V3 mg = {-g.x, -g.y, -g.z};
  AbaDown<TP> d;
  sfor<0, TP::N>([&](auto I_) __attribute__((always_inline)) {
    constexpr int I = decltype(I_)::value;
    if constexpr (TM::attach(W, I)) {
      const Frc a = get_frc(acc, 6 * cidx<TrunkRows<TP>::body(I)>);
      d.a[I] = {a.n, a.f};
      d.w[I] = s.w[I];
    } else if constexpr (TM::in(W, I)) {
      aba_down<TP, I>(tb, mg, s, d, q, qd, qdd);
    }
  });
}

// =================================================================== operational-space control
// One sweep over the factor (see osc_sweep_bias and osc_sweep_task, which on
// one lane are two: with all seven right-hand sides one lane spills). Right-hand
// side 0 is tau_null; 1 to 6 are the rows of J in E's axes and only exist on
// E's path. The wave that has E hands the trunk, besides its rows, its share of
// right-hand sides 1 to 6, of Lambda^-1 and of the task acceleration, and the
// transform that the path's next body needs.
template <class TP, int E>
struct OscRhs {
  static constexpr bool on(int r, int k) { return r == 0 || TP::is_anc(TP::body_of(k), E); }
};
template <class TP, int E>
struct OscRows {  // rows that the wave of E adds: y shares (6 a DoF), then G, a*, and A and o
  static constexpr int kWave = Team<TP>::kPlan.wave[E];  // -1: E is a trunk body
  static constexpr int yrow(int k) { return 6 * TrunkRows<TP>::row(k); }
  static constexpr int kG = 6 * TrunkRows<TP>::total(), kA = kG + 21, kT = kA + 6;
  static constexpr int total() { return kWave < 0 ? 0 : kT + 12; }
  // the trunk body that E's branch hangs on (-1: the world)
  static constexpr int anchor() {
    int i = E;
    while (i >= 0 && !Team<TP>::trunk(i)) i = TP::parent(i);
    return i;
  }
};

// What OSC adds to a sweep up: tau_null, and on E's path the task's
// right-hand sides and sums. tau(k, v) takes h + tau_null.
template <class TP, int E, class QD, class TGT, class TO>
struct OscHook {
  const float* t;
  const QD& qd;
  const TGT& tgt;
  const TO& tau;
  float kp, kd, kn;
  M3 Rw[TP::N];
  V3 pw[TP::N];
  M3 A = {{1.0f, 0.0f, 0.0f, 0.0f, 1.0f, 0.0f, 0.0f, 0.0f, 1.0f}};  // axes and origin of the next path
  V3 o = {0.0f, 0.0f, 0.0f};                                         // body to close, in E's frame
  float G[6][6], a[6];  // shares of Lambda^-1 and of a* - J M^-1 tau_null
  float col[TP::NV][6];  // J, by DoF
  RBD_DI void init() {
#pragma unroll
    for (int i = 0; i < 6; ++i) {
      a[i] = 0.0f;
#pragma unroll
      for (int j = 0; j < 6; ++j) G[i][j] = 0.0f;
    }
  }
  template <class I_, class ST>
  RBD_DI void motion(I_, const ST& s) {
    constexpr int I = I_::value;
    if constexpr (TP::is_anc(I, E)) {
      struct Q0 {
        const ST& s;
        RBD_DI float operator()(int c) const { return c == 0 ? s.p0.x : (c == 1 ? s.p0.y : s.p0.z); }
      };
      world_pose<TP, I>(t, Q0{s}, s.R[I], Rw, pw);
    }
    if constexpr (I == E) {
      float err[6];
      pose_error<TP, E>(t, Rw[E], pw[E], tgt, err);
      const V3 el = mulT(Rw[E], V3{err[0], err[1], err[2]}), ea = mulT(Rw[E], V3{err[3], err[4], err[5]});
      const float e6[6] = {el.x, el.y, el.z, ea.x, ea.y, ea.z};
      const float tw[6] = {s.v[E].v.x, s.v[E].v.y, s.v[E].v.z, s.v[E].w.x, s.v[E].w.y, s.v[E].w.z};
#pragma unroll
      for (int i = 0; i < 6; ++i) a[i] = a[i] + (kp * e6[i] - kd * tw[i]);
    }
  }
  template <class J_, class ST, int n>
  RBD_DI void sides(J_, int k, const ST& s, float (&b)[n]) {
    constexpr int J = J_::value;
    b[0] = -kn * qd(k);
    tau(k, s.f[J].n.z + b[0]);
    if constexpr (n > 1 && TP::is_anc(J, E)) {
      const V3 z = {A.a[2], A.a[5], A.a[8]};
      const V3 lin = cross(o, z);
      col[k][0] = lin.x; col[k][1] = lin.y; col[k][2] = lin.z;
      col[k][3] = z.x; col[k][4] = z.y; col[k][5] = z.z;
#pragma unroll
      for (int i = 0; i < 6; ++i) b[i + 1] = col[k][i];
    }
  }
  template <class ST, int n>
  RBD_DI void base_sides(int k, const ST& s, float (&b)[n]) {
    const float hb[6] = {s.f[0].f.x, s.f[0].f.y, s.f[0].f.z, s.f[0].n.x, s.f[0].n.y, s.f[0].n.z};
    b[0] = -kn * qd(k);
    tau(k, __builtin_fmaf(-kn, qd(k), hb[k]));
    if constexpr (n > 1 && TP::is_anc(0, E)) {  // (not where E's root stands beside the base)
      const int c = k % 3;
      const V3 ax = {A.a[c], A.a[3 + c], A.a[6 + c]};
      const V3 lin = k < 3 ? ax : cross(o, ax);
      col[k][0] = lin.x; col[k][1] = lin.y; col[k][2] = lin.z;
      col[k][3] = k < 3 ? 0.0f : ax.x; col[k][4] = k < 3 ? 0.0f : ax.y; col[k][5] = k < 3 ? 0.0f : ax.z;
#pragma unroll
      for (int i = 0; i < 6; ++i) b[i + 1] = col[k][i];
    }
  }
  template <class J_, class ST, int n>
  RBD_DI void closed(J_, const ST& s, const Ltl<TP, n>& F) {
    constexpr int J = J_::value;
    if constexpr (n > 1 && TP::is_anc(J, E)) {
      sfor<0, cidx<TP::nvb(J)>>([&](auto C_) __attribute__((always_inline)) {
        constexpr int k = TP::vofs(J) + decltype(C_)::value;
#pragma unroll
        for (int i = 0; i < 6; ++i) {
          a[i] = __builtin_fmaf(-F.y[i + 1][k], F.y[0][k], a[i]);
#pragma unroll
          for (int j = 0; j <= i; ++j) G[i][j] = __builtin_fmaf(F.y[i + 1][k], F.y[j + 1][k], G[i][j]);
        }
      });
      if constexpr (TP::parent(J) >= 0) {
        A = mulMMT(A, s.R[J]);
        o = o - mul(A, load_r<J>(t));
      }
    }
  }
  // J^T z of DoF k
  RBD_DI float task_torque(int k, const float (&z)[6]) const {
    float x = 0.0f;
#pragma unroll
    for (int i = 0; i < 6; ++i) x = __builtin_fmaf(col[k][i], z[i], x);
    return x;
  }
};

// The trunk's: takes the wave of E's share off right-hand sides 1 to 6.
template <class TP, int E, class H>
struct OscTrunkHook {
  using EROWS = OscRows<TP, E>;
  H& h;
  const LdsCol& ex;
  template <bool ON, int n>
  RBD_DI void share(int k, float (&b)[n]) {
    if constexpr (ON && EROWS::kWave >= 0) {
#pragma unroll
      for (int r = 0; r < 6; ++r) b[r + 1] = b[r + 1] - ex.get(EROWS::yrow(k) + r);
    }
  }
  template <class J, class ST, int n>
  RBD_DI void sides(J j, int k, const ST& s, float (&b)[n]) {
    h.sides(j, k, s, b);
    share<TP::is_anc(J::value, E)>(k, b);
  }
  template <class ST, int n>
  RBD_DI void base_sides(int k, const ST& s, float (&b)[n]) {
    h.base_sides(k, s, b);
    share<TP::is_anc(0, E)>(k, b);
  }
  template <class J, class ST, class LF>
  RBD_DI void closed(J j, const ST& s, const LF& F) {
    h.closed(j, s, F);
  }
};

}  // namespace rbd
