// HIP kernels for gfx950, templated on the tree type. Device code only, with
// no host headers: the ahead-of-time build instantiates it per compiled
// topology (rbd_kern_topo.hip) and the runtime compiler per new topology
// (rbd_jit.cpp), from the same text. The per-lane algorithms live in
// rbd_lane.hpp; kernel ids and launch shapes are chosen on the host
// (rbd_dispatch.cpp).
#pragma once

#include "rbd_lane.hpp"
#include "rbd_shared.hpp"
#include "rbd_team.hpp"

namespace rbd {

RBD_DI uint32_t lane_id() { return blockIdx.x * blockDim.x + threadIdx.x; }

// Views of outputs that a later sweep of the same kernel reads back: not
// restrict-qualified, so the compiler keeps every load before the store that
// later overwrites the same element.
template <bool SB>
struct InAliasT {
  const float* base;
  int64_t ld;
  uint32_t lane;
  RBD_DI float operator()(int c) const {
    if constexpr (SB) return *lane_ptr(base + c * ld, lane);
    else return (base + c * ld)[lane];
  }
};
template <bool SB>
struct OutAliasT {
  float* base;
  int64_t ld;
  uint32_t lane;
  RBD_DI void operator()(int c, float v) const {
    if constexpr (SB) *lane_ptr(base + c * ld, lane) = v;
    else (base + c * ld)[lane] = v;
  }
};
using InAlias = InAliasT<true>;
using OutAlias = OutAliasT<true>;
template <bool SB>
struct OutAliasPT : OutAliasT<SB> {
  using In = InAliasT<SB>;
};
using OutAliasP = OutAliasPT<true>;

// The lane I/O views of a tree's kernels (kScalarBase picks the address form).
#define RBD_LANE_IO(TP)                           \
  constexpr bool kSB_ = kScalarBase<TP>;          \
  using In = InT<kSB_>;                           \
  using Out = OutT<kSB_>;                         \
  using InAlias = InAliasT<kSB_>;                 \
  using OutAlias = OutAliasT<kSB_>;               \
  using OutAliasP = OutAliasPT<kSB_>;             \
  (void)kSB_

// Between two sweeps: keeps the scheduler from starting the next sweep's
// loads inside the previous one, where its registers are all in use.
RBD_DI void sweep_boundary() { __builtin_amdgcn_sched_barrier(0); }

// Registers of one lane holding a preloaded input vector.
struct RegView {
  const float* x;
  RBD_DI float operator()(int k) const { return x[k]; }
};
// Loads entries 0..n-1 of input views into registers.
template <int n, class A>
RBD_DI void preload_inputs(float (&x)[n], const A& a) {
  sfor<0, n>([&](auto K_) __attribute__((always_inline)) { x[decltype(K_)::value] = a(decltype(K_)::value); });
}
template <int n, class A, class B>
RBD_DI void preload_inputs(float (&x)[n], float (&y)[n], const A& a, const B& b) {
  sfor<0, n>([&](auto K_) __attribute__((always_inline)) {
    constexpr int K = decltype(K_)::value;
    x[K] = a(K);
    y[K] = b(K);
  });
}

// Where a tree runs an operation as a team at every batch (or, for the kernels
// of two waves per 64 instances, at every batch that they would run), the kernel
// of the operation below is never launched and left empty.
template <class TP, TeamOp OP, long long BATCH = kTeamEvery>
inline constexpr bool kLanes = Team<TP>::template kLimit<OP> < BATCH;

template <class TP>
__global__ __launch_bounds__(kBlock) void k_fk(const float* __restrict__ tab, int64_t batch, int64_t ld,
                                               const float* __restrict__ q, float* __restrict__ T) {
  RBD_LANE_IO(TP);
  const uint32_t b = lane_id();
  if (b >= batch) return;
  fk_lane<TP>(tab, In{q, ld, b}, OutNT{T, ld, b});
}

template <class TP>
__global__ __launch_bounds__(kBlock) void k_jacobian(const float* __restrict__ tab, int64_t batch, int64_t ld,
                                                     const float* __restrict__ q, JacSlots js,
                                                     float* __restrict__ J) {
  RBD_LANE_IO(TP);
  const uint32_t b = lane_id();
  if (b >= batch) return;
  jac_lane<TP>(tab, In{q, ld, b}, js, J, ld, b);
}

// EXT: per-body external forces (fext, [6 n][ld]) enter the force balance.
// PRE (no external forces): every input load is issued at entry, as in
// k_fwd_dyn.
// Two waves per SIMD for branched trees up to 36 DoFs, where the sweep comes near
// the 256 registers that leaves them (31 bodies: 259 of its own accord, then 45 us
// at batch 131072; 231 without a spill when told so; a chain of 36 would spill).
template <class TP, bool HAS_QDD, bool EXT, bool PRE = false>
__global__ __launch_bounds__(kBlock, (!EXT && Team<TP>::kOn && TP::NV <= 36 ? 2 : 1)) void k_rnea(
    const float* __restrict__ tab, int64_t batch, int64_t ld, const float* __restrict__ q,
    const float* __restrict__ qd, const float* __restrict__ qdd, const float* __restrict__ fext,
    float* __restrict__ tau) {
  if constexpr (kLanes<TP, TeamOp::kId>) {
    const uint32_t b = lane_id();
    if (b >= batch) return;
    if constexpr (PRE && !EXT) {
      constexpr int NQ = TP::NQ, NV = TP::NV;
      float qv[NQ], qdv[NV], qddv[NV];
      const In qi{q, ld, b}, qdi{qd, ld, b}, qddi{HAS_QDD ? qdd : qd, ld, b};
      sfor<0, NQ>([&](auto K_) __attribute__((always_inline)) { qv[decltype(K_)::value] = qi(decltype(K_)::value); });
      sfor<0, NV>([&](auto K_) __attribute__((always_inline)) {
        qdv[decltype(K_)::value] = qdi(decltype(K_)::value);
        if constexpr (HAS_QDD) qddv[decltype(K_)::value] = qddi(decltype(K_)::value);
      });
      rnea_lane<TP, HAS_QDD>(tab, RegView{qv}, RegView{qdv}, RegView{HAS_QDD ? qddv : qdv}, Out{tau, ld, b});
    } else if constexpr (EXT)
      rnea_lane<TP, HAS_QDD>(tab, In{q, ld, b}, In{qd, ld, b}, In{HAS_QDD ? qdd : q, ld, b}, Out{tau, ld, b},
                             FextIn{{fext, ld, b}});
    else
      rnea_lane<TP, HAS_QDD>(tab, In{q, ld, b}, In{qd, ld, b}, In{HAS_QDD ? qdd : q, ld, b}, Out{tau, ld, b});
  }
}

template <class TP>
__global__ __launch_bounds__(kBlock) void k_crba(const float* __restrict__ tab, int64_t batch, int64_t ld,
                                                 const float* __restrict__ q, float* __restrict__ M) {
  RBD_LANE_IO(TP);
  const uint32_t b = lane_id();
  if (b >= batch) return;
  crba_lane<TP>(tab, In{q, ld, b}, M, ld, b);
}

template <class X>
struct RhsOne {
  X tau;
  RBD_DI float operator()(int, int k) const { return tau(k); }
};
template <class Y>
struct SinkOne {
  Y x;
  RBD_DI void operator()(int, int k, float v) const { x(k, v); }
};

// PRE = true issues every input load of the lane at entry (106 for the
// humanoid), so their latency overlaps the first bodies' arithmetic instead of
// stalling the single wave of each SIMD at every body.
// The external-force view of a kernel: FextIn over fext, or nothing.
template <bool EXT>
RBD_DI auto fext_view(const float* fext, int64_t ld, uint32_t b) {
  if constexpr (EXT) return FextIn{{fext, ld, b}};
  else return NoFext{};
}

// EXT as for k_rnea.
template <class TP, bool PRE, bool EXT>
__global__ __launch_bounds__(kBlock) void k_fwd_dyn(const float* __restrict__ tab, int64_t batch, int64_t ld,
                                                    const float* __restrict__ q, const float* __restrict__ qd,
                                                    const float* __restrict__ tau, const float* __restrict__ fext,
                                                    float* __restrict__ qdd) {
  if constexpr (kLanes<TP, EXT ? TeamOp::kFdExt : TeamOp::kFd>) {
    const uint32_t b = lane_id();
    if (b >= batch) return;
    const auto fx = fext_view<EXT>(fext, ld, b);
    if constexpr (PRE) {
      constexpr int NQ = TP::NQ, NV = TP::NV;
      float qv[NQ], qdv[NV], tv[NV];
      const In qi{q, ld, b}, qdi{qd, ld, b}, ti{tau, ld, b};
      sfor<0, NQ>([&](auto K_) __attribute__((always_inline)) { qv[decltype(K_)::value] = qi(decltype(K_)::value); });
      sfor<0, NV>([&](auto K_) __attribute__((always_inline)) {
        qdv[decltype(K_)::value] = qdi(decltype(K_)::value);
        tv[decltype(K_)::value] = ti(decltype(K_)::value);
      });
      fwd_dyn_lane<TP, 1>(tab, RegView{qv}, RegView{qdv}, RhsOne<RegView>{RegView{tv}}, SinkOne<Out>{Out{qdd, ld, b}},
                          fx);
    } else {
      fwd_dyn_lane<TP, 1>(tab, In{q, ld, b}, In{qd, ld, b}, RhsOne<In>{In{tau, ld, b}}, SinkOne<Out>{Out{qdd, ld, b}},
                          fx);
    }
  }
}

// Forward dynamics by the articulated-body algorithm; PRE as for k_fwd_dyn,
// EXT as for k_rnea.
template <class TP, bool PRE, bool EXT>
__global__ __launch_bounds__(kBlock) void k_aba(const float* __restrict__ tab, int64_t batch, int64_t ld,
                                                const float* __restrict__ q, const float* __restrict__ qd,
                                                const float* __restrict__ tau, const float* __restrict__ fext,
                                                float* __restrict__ qdd) {
  if constexpr (kLanes<TP, EXT ? TeamOp::kFdExt : TeamOp::kFd>) {
    const uint32_t b = lane_id();
    if (b >= batch) return;
    const auto fx = fext_view<EXT>(fext, ld, b);
    if constexpr (PRE) {
      constexpr int NQ = TP::NQ, NV = TP::NV;
      float qv[NQ], qdv[NV], tv[NV];
      const In qi{q, ld, b}, qdi{qd, ld, b}, ti{tau, ld, b};
      sfor<0, NQ>([&](auto K_) __attribute__((always_inline)) { qv[decltype(K_)::value] = qi(decltype(K_)::value); });
      sfor<0, NV>([&](auto K_) __attribute__((always_inline)) {
        qdv[decltype(K_)::value] = qdi(decltype(K_)::value);
        tv[decltype(K_)::value] = ti(decltype(K_)::value);
      });
      aba_lane<TP>(tab, RegView{qv}, RegView{qdv}, RegView{tv}, Out{qdd, ld, b}, fx);
    } else {
      aba_lane<TP>(tab, In{q, ld, b}, In{qd, ld, b}, In{tau, ld, b}, Out{qdd, ld, b}, fx);
    }
  }
}

// ---- fwd_dyn adjoint: solve M [qdd, lam] = [tau - h, gbar] with one factor,
// write g_tau = lam, then run the inverse-dynamics adjoint at (q, qd, qdd).
template <class X>
struct RhsTwo {
  X tau, gbar;
  RBD_DI float operator()(int r, int k) const { return r == 0 ? tau(k) : gbar(k); }
};
struct SinkRegs {
  float* qdd;
  float* lam;
  RBD_DI void operator()(int r, int k, float v) const {
    if (r == 0) qdd[k] = v; else lam[k] = v;
  }
};
// An output that may be absent (null base).
template <class Y>
struct OutOpt {
  Y y;
  bool on;
  RBD_DI void operator()(int c, float v) const {
    if (on) y(c, v);
  }
};
// q-double-dot and lam parked in the g_qd and g_tau outputs go through the
// alias views above.
template <class Y>
struct SinkTwo {
  Y qdd, lam;
  RBD_DI void operator()(int r, int k, float v) const {
    if (r == 0) qdd(k, v); else lam(k, v);
  }
};
// A per-lane row parked in LDS: entry c of lane l of a wave at
// p[c * 64 + l] (consecutive lanes in consecutive banks; the entry offset is
// a compile-time immediate).
struct LdsRow {
  float* p;
  RBD_DI void operator()(int c, float v) const { p[c * kTileLanes] = v; }
  struct In {
    const float* p;
    RBD_DI float operator()(int c) const { return p[c * kTileLanes]; }
  };
};

template <class TP, bool ADJ, class QI, class X, class GQ, class GQD, class GT, class FX = NoFext, class GF = NoGF>
RBD_DI void vjp_lane(const float* __restrict__ tab, const QI& q, const X& qd, const X& tau, const X& gqdd,
                     const GQ& gq, const GQD& gqd, const GT& gtau, const FX& fx = FX{}, const GF& gf = GF{}) {
  constexpr int NV = TP::NV;
  float qddv[NV], lam[NV];
  fwd_dyn_lane<TP, 2>(tab, q, qd, RhsTwo<X>{tau, gqdd}, SinkRegs{qddv, lam}, fx);
  sfor<0, NV>([&](auto K_) __attribute__((always_inline)) {
    constexpr int K = decltype(K_)::value;
    gtau(K, lam[K]);
  });
  if constexpr (ADJ) id_adjoint_lane<TP>(tab, q, qd, RegView{qddv}, RegView{lam}, gq, gqd, fx, gf);
}

// q-double-dot parked in g_qd and lam in g_tau between the solve and the
// adjoint sweep, instead of 2 nv registers held across it. Every element is
// read by its body's forward step before that body's backward step
// overwrites g_qd.
template <class TP, class QI, class X, class GQ, class P, class FX = NoFext, class GF = NoGF>
RBD_DI void vjp_lane_parked(const float* __restrict__ tab, const QI& q, const X& qd, const X& tau, const X& gqdd,
                            const GQ& gq, const P& gqd_out, const P& gtau_out, const typename P::In& gqd_in,
                            const typename P::In& gtau_in, const FX& fx = FX{}, const GF& gf = GF{}) {
  fwd_dyn_lane<TP, 2>(tab, q, qd, RhsTwo<X>{tau, gqdd}, SinkTwo<P>{gqd_out, gtau_out}, fx);
  id_adjoint_lane<TP>(tab, q, qd, gqd_in, gtau_in, gq, gqd_out, fx, gf);
}

struct RowAlias {
  GlobalF* p;
  RBD_DI RowAlias(float* q) : p((GlobalF*)q) {}
  RBD_DI void operator()(int c, float v) const { p[c] = v; }
  struct In {
    const GlobalF* p;
    RBD_DI In(const float* q) : p((const GlobalF*)q) {}
    RBD_DI float operator()(int c) const { return p[c]; }
  };
};

// MODE 0: g_tau only; 1: adjoint with q-double-dot and lam in registers (some
// output absent); 2: adjoint with both parked in g_qd and g_tau (both
// requested); 3 (large trees, any outputs): both parked in LDS (dynamic shared
// memory, 2 NV floats per lane), the adjoint on fresh views. EXT (modes 1 to
// 3): external forces fext (nullable: zero) in the dynamics and the force
// cotangent g_fext (nullable).
// Two waves per SIMD for branched trees of 17 and 18 DoFs, where the two sweeps
// come near the 256 registers that leaves them (18 DoFs: 256 and 265 of their own
// accord, and with 265 45.1 us at batch 98304 against 36.4).
template <class TP, int MODE, bool EXT = false>
__global__ __launch_bounds__(kBlock, (!EXT && MODE == 3 && Team<TP>::kOn && TP::NV <= 18 ? 2 : 1)) void k_fwd_dyn_vjp(
    const float* __restrict__ tab, int64_t batch, int64_t ld, const float* __restrict__ q,
    const float* __restrict__ qd, const float* __restrict__ tau, const float* __restrict__ gqdd, float* gq, float* gqd,
    float* gtau, const float* __restrict__ fext, float* gfext) {
  if constexpr (MODE == 0 || kLanes<TP, EXT ? TeamOp::kVjpExt : TeamOp::kVjp>) {
    static_assert(!EXT || MODE >= 1, "external forces: modes 1 to 3");
    RBD_LANE_IO(TP);
    const uint32_t b = lane_id();
    if (b >= batch) return;
    const In qi{q, ld, b}, qdi{qd, ld, b}, ti{tau, ld, b}, gi{gqdd, ld, b};
    const OutOpt<OutAlias> gqo{OutAlias{gq, ld, b}, gq != nullptr};
    // the external-force views (nothing without EXT)
    auto fx_view = [&](const float* p, int64_t l) __attribute__((always_inline)) {
      if constexpr (EXT) return FextOpt{{p, l, b}};
      else return NoFext{};
    };
    auto gf_view = [&](int64_t l) __attribute__((always_inline)) {
      if constexpr (EXT) return GFOut{{gfext, l, b}};
      else return NoGF{};
    };
    if constexpr (MODE == 3) {
      // the two sweeps, the second on fresh views (its own table and input
      // pointers and row stride): a large tree's first sweep uses every
      // register, and values kept for the second one spill (measured: 1028 ->
      // 400 B/lane of scratch, 126 -> 108 us for the humanoid). Each wave parks
      // in its region of the block's dynamic LDS: [qdd rows | lam rows].
      extern __shared__ float lds_park[];
      constexpr int NV = TP::NV;
      float* const w = lds_park + (threadIdx.x / kTileLanes) * (2 * NV * kTileLanes) + (threadIdx.x % kTileLanes);
      fwd_dyn_lane<TP, 2>(tab, qi, qdi, RhsTwo<In>{ti, gi}, SinkTwo<LdsRow>{LdsRow{w}, LdsRow{w + NV * kTileLanes}},
                          fx_view(fext, ld));
      if (gtau) {
        sfor<0, NV>([&](auto K_) __attribute__((always_inline)) {
          constexpr int K = decltype(K_)::value;
          Out{gtau, ld, b}(K, w[(NV + K) * kTileLanes]);
        });
      }
      sweep_boundary();
      const int64_t l2 = opaque(ld);
      // (issuing this sweep's q and qd loads at its start cut the spill from 536
      // to 24 B/lane but measured 79.2 against 77.0 us for the humanoid at 32768)
      id_adjoint_lane<TP>(opaque_table(tab), In{opaque(q), l2, b}, In{opaque(qd), l2, b}, LdsRow::In{w},
                          LdsRow::In{w + NV * kTileLanes}, OutOpt<OutAlias>{OutAlias{gq, l2, b}, gq != nullptr},
                          OutOpt<OutAlias>{OutAlias{gqd, l2, b}, gqd != nullptr}, fx_view(opaque(fext), l2),
                          gf_view(l2));
    } else if constexpr (MODE == 2) {
      const OutAliasP pd{{gqd, ld, b}}, pt{{gtau, ld, b}};
      vjp_lane_parked<TP>(tab, qi, qdi, ti, gi, gqo, pd, pt, InAlias{gqd, ld, b}, InAlias{gtau, ld, b},
                          fx_view(fext, ld), gf_view(ld));
    } else {
      vjp_lane<TP, MODE == 1>(tab, qi, qdi, ti, gi, gqo, OutOpt<OutAlias>{OutAlias{gqd, ld, b}, gqd != nullptr},
                              OutOpt<OutAlias>{OutAlias{gtau, ld, b}, gtau != nullptr}, fx_view(fext, ld),
                              gf_view(ld));
    }
  }
}

// ---- the adjoint on two waves per 64 instances (a block of 128 lanes), for
// large trees at batches small enough that one wave per 64 instances leaves
// SIMDs idle: wave 0 solves for qdd (the fused sweep) while wave 1 factors M
// on its own and solves lam = M^-1 g_qdd (the bias-free sweep; g_tau = lam).
// Nothing but qdd and lam crosses the block's one barrier, parked in LDS
// ([qdd rows | lam rows], 64 lanes each); then wave 0 runs the adjoint sweep
// on fresh views. Every lane of the block reaches the barrier.
template <class TP, bool EXT = false>
__global__ __launch_bounds__(2 * kTileLanes) void k_fwd_dyn_vjp_split(
    const float* __restrict__ tab, int64_t batch, int64_t ld, const float* __restrict__ q,
    const float* __restrict__ qd, const float* __restrict__ tau, const float* __restrict__ gqdd, float* gq,
    float* gqd, float* gtau, const float* __restrict__ fext, float* gfext) {
  if constexpr (kLanes<TP, EXT ? TeamOp::kVjpExt : TeamOp::kVjp, kHalfWavePerSimd>) {
    RBD_LANE_IO(TP);
    constexpr int NQ = TP::NQ, NV = TP::NV;
    extern __shared__ float lds_vjp[];
    const uint32_t lane = threadIdx.x % kTileLanes;
    const bool solver = threadIdx.x >= kTileLanes;
    const uint32_t b = blockIdx.x * kTileLanes + lane;
    const bool valid = b < batch;
    float* const qpark = lds_vjp + lane;
    float* const lpark = lds_vjp + NV * kTileLanes + lane;
    auto fx_view = [&](const float* p, int64_t l) __attribute__((always_inline)) {
      if constexpr (EXT) return FextOpt{{p, l, b}};
      else return NoFext{};
    };
    auto gf_view = [&](int64_t l) __attribute__((always_inline)) {
      if constexpr (EXT) return GFOut{{gfext, l, b}};
      else return NoGF{};
    };
    if (!solver) {
      if (valid) {
        if constexpr (EXT) {
          fwd_dyn_lane<TP, 1>(tab, In{q, ld, b}, In{qd, ld, b}, RhsOne<In>{In{tau, ld, b}},
                              SinkOne<LdsRow>{LdsRow{qpark}}, fx_view(fext, ld));
        } else {
          // every input load at entry, as in k_fwd_dyn for large trees
          float qv[NQ], qdv[NV], tv[NV];
          preload_inputs<NQ>(qv, In{q, ld, b});
          preload_inputs<NV>(qdv, tv, In{qd, ld, b}, In{tau, ld, b});
          fwd_dyn_lane<TP, 1>(tab, RegView{qv}, RegView{qdv}, RhsOne<RegView>{RegView{tv}},
                              SinkOne<LdsRow>{LdsRow{qpark}});
        }
      }
    } else if (valid) {
      fwd_dyn_lane<TP, 1, In, In, RhsOne<In>, SinkOne<LdsRow>, NoFext, false>(
          tab, In{q, ld, b}, In{qd, ld, b}, RhsOne<In>{In{gqdd, ld, b}}, SinkOne<LdsRow>{LdsRow{lpark}});
      if (gtau) {
        sfor<0, NV>([&](auto K_) __attribute__((always_inline)) {
          constexpr int K = decltype(K_)::value;
          Out{gtau, ld, b}(K, lpark[K * kTileLanes]);
        });
      }
    }
    __syncthreads();
    if (!solver && valid) {
      sweep_boundary();
      const int64_t l2 = opaque(ld);
      id_adjoint_lane<TP>(opaque_table(tab), In{opaque(q), l2, b}, In{opaque(qd), l2, b}, LdsRow::In{qpark},
                          LdsRow::In{lpark}, OutOpt<OutAlias>{OutAlias{gq, l2, b}, gq != nullptr},
                          OutOpt<OutAlias>{OutAlias{gqd, l2, b}, gqd != nullptr}, fx_view(opaque(fext), l2),
                          gf_view(l2));
    }
  }
}

// ---- fwd_dyn tangent, three sweeps of one lane: qdd by the fused solve
// (parked in the qdd output when one is given, else in dqdd), the tangent of
// inverse dynamics writing dtau - d(ID) into dqdd, and the solve with M in
// place (each right-hand-side entry is read when its subtree closes, every
// result written after the sweep). Neither output is restrict-qualified, so
// loads of parked values stay ordered with the stores.
// EXT: external forces fext and their tangent dfext (each nullable: zero).
template <class TP, bool EXT = false>
__global__ __launch_bounds__(kBlock) void k_fwd_dyn_jvp(const float* __restrict__ tab, int64_t batch, int64_t ld,
                                                        const float* __restrict__ q, const float* __restrict__ qd,
                                                        const float* __restrict__ tau, const float* __restrict__ dq,
                                                        const float* __restrict__ dqd,
                                                        const float* __restrict__ dtau, float* qdd, float* dqdd,
                                                        const float* __restrict__ fext,
                                                        const float* __restrict__ dfext) {
  if constexpr (kLanes<TP, TeamOp::kJvp>) {
    RBD_LANE_IO(TP);
    const uint32_t b = lane_id();
    if (b >= batch) return;
    float* park = qdd ? qdd : dqdd;
    auto fx_view = [&](const float* p, int64_t l) __attribute__((always_inline)) {
      if constexpr (EXT) return FextOpt{{p, l, b}};
      else return NoFext{};
    };
    // a large tree, and any with forces, gives each sweep fresh views (see
    // k_fwd_dyn_vjp) and with forces keeps the sweeps apart (7 joints at batch
    // 262144: 94.8 -> 84.0 us, 1307 -> 660 spilled scalars moved)
    constexpr bool kFresh = TP::NV > 16 || EXT;
    fwd_dyn_lane<TP, 1>(tab, In{q, ld, b}, In{qd, ld, b}, RhsOne<In>{In{tau, ld, b}},
                        SinkOne<OutAlias>{OutAlias{park, ld, b}}, fx_view(fext, ld));
    if constexpr (EXT) sweep_boundary();
    auto view = [](auto x) __attribute__((always_inline)) {
      if constexpr (kFresh) return opaque(x);
      else return x;
    };
    auto view_table = [](const float* x) __attribute__((always_inline)) {
      if constexpr (kFresh) return opaque_table(x);
      else return x;
    };
    const int64_t ld2 = view(ld);
    if constexpr (kFresh && !EXT) {
      // every input load of the tangent sweep issued at its start, as in k_rnea_jvp
      constexpr int NQ = TP::NQ, NV = TP::NV;
      float qv[NQ], qdv[NV], dqv[NQ], dqdv[NV], dtv[NV];
      preload_inputs<NQ>(qv, dqv, In{view(q), ld2, b}, In{dq, ld2, b});
      preload_inputs<NV>(qdv, dqdv, In{view(qd), ld2, b}, In{dqd, ld2, b});
      preload_inputs<NV>(dtv, In{dtau, ld2, b});
      id_tangent_lane<TP>(view_table(tab), RegView{qv}, RegView{qdv}, InAlias{park, ld2, b}, RegView{dqv},
                          RegView{dqdv}, RegView{dtv}, OutAlias{dqdd, ld2, b});
    } else {
      id_tangent_lane<TP>(view_table(tab), In{view(q), ld2, b}, In{view(qd), ld2, b}, InAlias{park, ld2, b},
                          In{dq, ld2, b}, In{dqd, ld2, b}, In{dtau, ld2, b}, OutAlias{dqdd, ld2, b},
                          fx_view(fext, ld2), fx_view(dfext, ld2));
    }
    if constexpr (EXT) sweep_boundary();
    const int64_t ld3 = view(ld2);
    fwd_dyn_lane<TP, 1, In, In, RhsOne<InAlias>, SinkOne<OutAlias>, NoFext, false>(
        view_table(tab), In{view(q), ld3, b}, In{qd, ld3, b}, RhsOne<InAlias>{InAlias{dqdd, ld3, b}},
        SinkOne<OutAlias>{OutAlias{dqdd, ld3, b}});
  }
}

// ---- the same tangent on two waves per 64 instances (a block of 128 lanes),
// for batches small enough that one wave per 64 instances leaves SIMDs idle:
// wave 0 runs the fused solve for qdd and the tangent of inverse dynamics and
// hands the right-hand side to wave 1 through LDS; wave 1 factors M in the
// meantime, then solves with it. Dynamic LDS per block: [rhs rows | qdd rows],
// 64 lanes each. Every lane of the block reaches the one barrier.
template <class TP, bool EXT = false>
__global__ __launch_bounds__(2 * kTileLanes) void k_fwd_dyn_jvp_split(
    const float* __restrict__ tab, int64_t batch, int64_t ld, const float* __restrict__ q,
    const float* __restrict__ qd, const float* __restrict__ tau, const float* __restrict__ dq,
    const float* __restrict__ dqd, const float* __restrict__ dtau, float* qdd, float* dqdd,
    const float* __restrict__ fext, const float* __restrict__ dfext) {
  if constexpr (kLanes<TP, TeamOp::kJvp, kHalfWavePerSimd>) {
    RBD_LANE_IO(TP);
    constexpr int NV = TP::NV;
    extern __shared__ float lds_jvp[];
    const uint32_t lane = threadIdx.x % kTileLanes;
    const bool solver = threadIdx.x >= kTileLanes;
    const uint32_t b = blockIdx.x * kTileLanes + lane;
    const bool valid = b < batch;
    float* const rhs = lds_jvp + lane;
    float* const qpark = lds_jvp + NV * kTileLanes + lane;
    auto fx_view = [&](const float* p, int64_t l) __attribute__((always_inline)) {
      if constexpr (EXT) return FextOpt{{p, l, b}};
      else return NoFext{};
    };
    Ltl<TP, 1> F;
    if (!solver) {
      if (valid) {
        fwd_dyn_lane<TP, 1>(tab, In{q, ld, b}, In{qd, ld, b}, RhsOne<In>{In{tau, ld, b}},
                            SinkOne<LdsRow>{LdsRow{qpark}}, fx_view(fext, ld));
        if (qdd) {
          sfor<0, NV>([&](auto K_) __attribute__((always_inline)) {
            constexpr int K = decltype(K_)::value;
            Out{qdd, ld, b}(K, qpark[K * kTileLanes]);
          });
        }
        sweep_boundary();
        const int64_t l2 = opaque(ld);
        if constexpr (!EXT) {
          // every input load of the tangent sweep issued at its start, as in k_rnea_jvp
          constexpr int NQ = TP::NQ;
          float qv[NQ], qdv[NV], dqv[NQ], dqdv[NV], dtv[NV];
          preload_inputs<NQ>(qv, dqv, In{opaque(q), l2, b}, In{dq, l2, b});
          preload_inputs<NV>(qdv, dqdv, In{opaque(qd), l2, b}, In{dqd, l2, b});
          preload_inputs<NV>(dtv, In{dtau, l2, b});
          id_tangent_lane<TP>(opaque_table(tab), RegView{qv}, RegView{qdv}, LdsRow::In{qpark}, RegView{dqv},
                              RegView{dqdv}, RegView{dtv}, LdsRow{rhs});
        } else {
          id_tangent_lane<TP>(opaque_table(tab), In{opaque(q), l2, b}, In{opaque(qd), l2, b}, LdsRow::In{qpark},
                              In{dq, l2, b}, In{dqd, l2, b}, In{dtau, l2, b}, LdsRow{rhs}, fx_view(opaque(fext), l2),
                              fx_view(opaque(dfext), l2));
        }
      }
    } else if (valid) {
      ltl_factor_lane<TP>(tab, In{q, ld, b}, F);
    }
    __syncthreads();
    if (solver && valid) {
      ltl_solve_y<TP>(F, LdsRow::In{rhs});
      ltl_back<TP, 1>(F, [&](int, int k, float v) __attribute__((always_inline)) { Out{dqdd, ld, b}(k, v); });
    }
  }
}

// ---- tangent of inverse dynamics, Eq. (1), along (dq, dqd, dqdd[, dF]): one
// sweep of id_tangent_lane with the acceleration tangent; the sweep writes
// 0 - d(ID), stored negated as d(ID) (both steps exact).
template <class V>
struct On : V {  // a view whose entries are used (kOn)
  static constexpr bool kOn = true;
};
template <class O>
struct Neg {  // an output written negated
  O o;
  static constexpr bool kOn = true;
  RBD_DI void operator()(int c, float v) const { o(c, -v); }
};

// PRE (no external forces): every input load is issued at entry, as in
// k_fwd_dyn.
template <class TP, bool EXT = false, bool PRE = false>
__global__ __launch_bounds__(kBlock) void k_rnea_jvp(const float* __restrict__ tab, int64_t batch, int64_t ld,
                                                     const float* __restrict__ q, const float* __restrict__ qd,
                                                     const float* __restrict__ qdd, const float* __restrict__ dq,
                                                     const float* __restrict__ dqd, const float* __restrict__ dqdd,
                                                     float* __restrict__ dtau, const float* __restrict__ fext,
                                                     const float* __restrict__ dfext) {
  if constexpr (kLanes<TP, EXT ? TeamOp::kIdJvpExt : TeamOp::kIdJvp>) {
    RBD_LANE_IO(TP);
    const uint32_t b = lane_id();
    if (b >= batch) return;
    auto fx_view = [&](const float* p) __attribute__((always_inline)) {
      if constexpr (EXT) return FextOpt{{p, ld, b}};
      else return NoFext{};
    };
    if constexpr (PRE && !EXT) {
      constexpr int NQ = TP::NQ, NV = TP::NV;
      float qv[NQ], qdv[NV], qddv[NV], dqv[NQ], dqdv[NV], dqddv[NV];
      const In qi{q, ld, b}, qdi{qd, ld, b}, qddi{qdd, ld, b}, dqi{dq, ld, b}, dqdi{dqd, ld, b}, dqddi{dqdd, ld, b};
      sfor<0, NQ>([&](auto K_) __attribute__((always_inline)) {
        constexpr int K = decltype(K_)::value;
        qv[K] = qi(K);
        dqv[K] = dqi(K);
      });
      sfor<0, NV>([&](auto K_) __attribute__((always_inline)) {
        constexpr int K = decltype(K_)::value;
        qdv[K] = qdi(K);
        qddv[K] = qddi(K);
        dqdv[K] = dqdi(K);
        dqddv[K] = dqddi(K);
      });
      id_tangent_lane<TP>(tab, RegView{qv}, RegView{qdv}, RegView{qddv}, RegView{dqv}, RegView{dqdv}, NoFext{},
                          Neg<Out>{Out{dtau, ld, b}}, NoFext{}, NoFext{}, On<RegView>{RegView{dqddv}});
    } else {
      id_tangent_lane<TP>(tab, In{q, ld, b}, In{qd, ld, b}, In{qdd, ld, b}, In{dq, ld, b}, In{dqd, ld, b}, NoFext{},
                          Neg<Out>{Out{dtau, ld, b}}, fx_view(fext), fx_view(dfext), On<In>{In{dqdd, ld, b}});
    }
  }
}

// ---- adjoint of inverse dynamics, Eq. (1), for the cotangent lam: one sweep
// of id_adjoint_lane at the given qdd. That sweep writes the cotangents of
// forward dynamics, -lam^T dID/d(q, qd) and J_i lam, which are stored negated
// (exact), and g_qdd = M lam. Every output may be absent (null).
template <class TP, bool EXT = false>
__global__ __launch_bounds__(kBlock) void k_rnea_vjp(const float* __restrict__ tab, int64_t batch, int64_t ld,
                                                     const float* __restrict__ q, const float* __restrict__ qd,
                                                     const float* __restrict__ qdd, const float* __restrict__ lam,
                                                     float* __restrict__ gq, float* __restrict__ gqd,
                                                     float* __restrict__ gqdd, const float* __restrict__ fext,
                                                     float* __restrict__ gfext) {
  if constexpr (kLanes<TP, EXT ? TeamOp::kIdVjpExt : TeamOp::kIdVjp>) {
    RBD_LANE_IO(TP);
    const uint32_t b = lane_id();
    if (b >= batch) return;
    auto opt = [&](float* p) __attribute__((always_inline)) { return OutOpt<Out>{Out{p, ld, b}, p != nullptr}; };
    auto fx_view = [&]() __attribute__((always_inline)) {
      if constexpr (EXT) return FextOpt{{fext, ld, b}};
      else return NoFext{};
    };
    auto gf_view = [&]() __attribute__((always_inline)) {
      if constexpr (EXT) return Neg<GFOut>{GFOut{{gfext, ld, b}}};
      else return NoGF{};
    };
    if constexpr (TP::NV > 16 && !EXT) {
      // every input load issued at entry, as in k_rnea_jvp
      constexpr int NQ = TP::NQ, NV = TP::NV;
      float qv[NQ], qdv[NV], qddv[NV], lv[NV];
      preload_inputs<NQ>(qv, In{q, ld, b});
      preload_inputs<NV>(qdv, qddv, In{qd, ld, b}, In{qdd, ld, b});
      preload_inputs<NV>(lv, In{lam, ld, b});
      id_adjoint_lane<TP>(tab, RegView{qv}, RegView{qdv}, RegView{qddv}, RegView{lv}, Neg<OutOpt<Out>>{opt(gq)},
                          Neg<OutOpt<Out>>{opt(gqd)}, NoFext{}, NoGF{}, On<OutOpt<Out>>{opt(gqdd)});
    } else {
      id_adjoint_lane<TP>(tab, In{q, ld, b}, In{qd, ld, b}, In{qdd, ld, b}, In{lam, ld, b}, Neg<OutOpt<Out>>{opt(gq)},
                          Neg<OutOpt<Out>>{opt(gqd)}, fx_view(), gf_view(), On<OutOpt<Out>>{opt(gqdd)});
    }
  }
}

// ---- controller workloads for one frame E: the last body (a leaf) ahead of
// time, any other body compiled at run time on its first use.
template <class TP, int E = TP::N - 1>
__global__ __launch_bounds__(kBlock) void k_diff_ik(const float* __restrict__ tab, int64_t batch, int64_t ld,
                                                    const float* __restrict__ q, const float* __restrict__ tgt,
                                                    float gain, float lam2, float* __restrict__ qd) {
  RBD_LANE_IO(TP);
  const uint32_t b = lane_id();
  if (b >= batch) return;
  diff_ik_lane<TP, E>(tab, In{q, ld, b}, In{tgt, ld, b}, gain, lam2, Out{qd, ld, b});
}

// =================================================================== teams of waves
// The kernels of a team (rbd_team.hpp): a block is one team, 64 instances, all
// lanes reach every barrier (lanes past the batch redo its last instance and
// store the same values to it).

// Entry c of an input or of LDS rows: of the wave's branches from `br` (moved),
// of the trunk from `tk`. DOF as for team_load.
template <class TP, bool DOF, class B, class T>
struct TeamView {
  B br;
  T tk;
  RBD_DI float operator()(int c) const {
    const int i = DOF ? TP::body_of(c) : (TP::kFree ? (c < 7 ? 0 : c - 6) : c);
    return Team<TP>::trunk(i) ? tk(c) : br(c);
  }
};
template <class TP, bool DOF, class I>
RBD_DI TeamView<TP, DOF, I, I> team_in(const float* p, int64_t off, int64_t ld, uint32_t b) {
  return {I{p + off, ld, b}, I{p, ld, b}};
}

// The team's external-force views: of the calling wave's branches and of the trunk.
template <bool EXT>
RBD_DI auto team_fext(const float* fext, int64_t ld, int shift, uint32_t b) {
  return fext_view<EXT>(fext + 6 * shift * ld, ld, b);
}
// The same where the forces may be absent (null: zero).
template <bool EXT>
RBD_DI auto team_fext_opt(const float* fext, int64_t ld, int shift, uint32_t b) {
  if constexpr (EXT) return FextOpt{{fext ? fext + 6 * shift * ld : nullptr, ld, b}};
  else return NoFext{};
}

// Where a team finds the arrays of its instances: structure-of-arrays batches,
// or one instance per row of N (the serving runtime's requests). `shift` bodies
// further on for branches.
template <class TP>
struct SoaIo {
  using I = InT<kScalarBase<TP>>;
  using O = OutT<kScalarBase<TP>>;
  int64_t ld;
  template <int N>
  RBD_DI I in(const float* p, int shift, uint32_t b) const {
    return {p + shift * ld, ld, b};
  }
  template <int N>
  RBD_DI O out(float* p, int shift, uint32_t b) const {
    return {p + shift * ld, ld, b};
  }
  // an output that may be absent
  template <int N>
  RBD_DI OutOpt<O> opt(float* p, int shift, uint32_t b) const {
    return {{p ? p + shift * ld : nullptr, ld, b}, p != nullptr};
  }
  RBD_DI SoaIo fresh() const { return {opaque(ld)}; }
};
struct RowIo {
  using I = InRow;
  using O = OutRow;
  template <int N>
  RBD_DI I in(const float* p, int shift, uint32_t b) const {
    return I(p + (int64_t)b * N + shift);
  }
  template <int N>
  RBD_DI O out(float* p, int shift, uint32_t b) const {
    return O(p + (int64_t)b * N + shift);
  }
  template <int N>
  RBD_DI O opt(float* p, int shift, uint32_t b) const {
    return out<N>(p, shift, b);
  }
  RBD_DI RowIo fresh() const { return {}; }
};
// Role W's entries of an input (above: of the trunk bodies above them too; the
// owner: of the whole trunk).
template <class TP, int W, bool ABOVE, bool DOF, class IO, int n>
RBD_DI void team_read(float (&x)[n], const IO& io, const float* p, const TeamLane& tl, bool owner) {
  constexpr int N = DOF ? TP::NV : TP::NQ;
  const auto tk = io.template in<N>(p, 0, tl.b);
  team_load<TP, W, ABOVE, DOF>(x, io.template in<N>(p, tl.shift, tl.b), tk);
  if constexpr (Team<TP>::may_own(W)) {
    if (owner) team_load_trunk<TP, DOF>(x, tk);
  }
}

// Rows of LDS of the blocks below.
template <class TP>
struct TeamLds {
  using Aba = TeamRows<TP, 27, false, 0>;
  using Fd2 = TeamRows<TP, 16, true, 2>;
  using Id = TeamRows<TP, 6, false, 0>;
  template <bool EXT>
  using Adj = TeamRows<TP, EXT ? 30 : 18, false, 0>;
  static constexpr int kAba = Aba::total() + 6 * TrunkRows<TP>::body(TP::N);  // and the trunk's accelerations
  static constexpr int kId = Id::total();
  // the solve's rows, which afterwards hold [qdd | lam | what the adjoint hands to the trunk], then x
  template <bool EXT>
  static constexpr int vjp_rows() {
    const int adj = 2 * TP::NV + Adj<EXT>::total();
    return Fd2::total() > adj ? Fd2::total() : adj;
  }
  template <bool EXT>
  static constexpr int vjp() {
    return vjp_rows<EXT>() + 2 * TrunkRows<TP>::total();
  }
};

// Forward dynamics of the calling wave's 64 instances, by the articulated-body
// algorithm for either entry point: branches up, the trunk up and down, branches
// down. Shared out over a team it needs half of the L^T L form's hand-over
// (27 rows of LDS per trunk body that carries branches against 16 and the trunk's
// rows of the factor: 108 against 226 for the humanoid)
// and few enough registers (168) for three waves per SIMD, and it is the more
// accurate of the two (humanoid: 1.7e-7 against 1.0e-6 in the Frobenius norm,
// 2.5e-7 against 5.7e-7 with contact forces). Bound: the longest branch's and
// the trunk's chain of vector instructions while the batch leaves SIMDs idle,
// their issue rate after that. Humanoid, against one lane per instance (L^T L):
// 33.8 -> 11.5 us at batch 64, 34.9 -> 12.7 at 16384, 37.2 -> 17.4 at 32768, 39.5 ->
// 26.4 at 65536, 88 -> 47.6 at 131072; the L^T L form as a team took 13.7, 15.0,
// 20.7, 34.5 and 64.9.
template <class TP, bool EXT, int W, class IO>
RBD_DI void team_aba(const TeamLane& tl, const float* __restrict__ tab, const IO& io, float* lds_rows, const float* q,
                     const float* qd, const float* tau, const float* fext, int64_t ld, float* qdd) {
  using TM = Team<TP>;
  using ROWS = typename TeamLds<TP>::Aba;
  constexpr int NQ = TP::NQ, NV = TP::NV;
  const LdsCol lds{lds_rows + tl.lane}, acc = lds.at(ROWS::total());
  const bool owner = TM::may_own(W) && tl.wave == TM::kOwner;
  const float* const t = opaque_table(tab);
  const float* const tb = opaque_table(tab + tl.shift * kBodyStride);
  float qv[NQ], qdv[NV], tv[NV];
  team_read<TP, W, true, false>(qv, io, q, tl, owner);
  team_read<TP, W, true, true>(qdv, io, qd, tl, owner);
  team_read<TP, W, false, true>(tv, io, tau, tl, owner);
  const RegView qr{qv}, qdr{qdv}, tr{tv};
  const auto fx = team_fext<EXT>(fext, ld, 0, tl.b);
  using FX = std::decay_t<decltype(fx)>;
  AbaState<TP, EXT> s;
  team_aba_up<TP, W, ROWS>(t, tb, s, qr, qdr, tr, team_fext<EXT>(fext, ld, tl.shift, tl.b),
                           lds.at(team_base<TP, ROWS, W>(tl)));
  if constexpr (TM::may_own(W)) {
    if (owner) {
      sfor<0, TP::N>([&](auto I_) __attribute__((always_inline)) {
        constexpr int I = decltype(I_)::value;
        // (those above its branches have their motion, but the forces were read with the moved view)
        if constexpr (TM::trunk(I) && (EXT || !TM::above(W, I))) aba_motion<TP, I>(t, s, qr, qdr, fx);
      });
    }
  }
  __syncthreads();
  if constexpr (TM::may_own(W)) {
    if (owner) team_aba_trunk<TP, ROWS, FX>(t, s, qr, qdr, tr, lds, acc, io.template out<NV>(qdd, 0, tl.b));
  }
  __syncthreads();
  team_aba_down<TP, W>(opaque_table(t), opaque_table(tb), s, qr, qdr, acc, io.template out<NV>(qdd, tl.shift, tl.b));
}

template <class TP, bool EXT>
__global__ __launch_bounds__(Team<TP>::kThreads, EXT ? 2 : 3) void k_aba_team(
    const float* __restrict__ tab, int64_t batch, int64_t ld, const float* __restrict__ q,
    const float* __restrict__ qd, const float* __restrict__ tau, const float* __restrict__ fext,
    float* __restrict__ qdd) {
  if constexpr (Team<TP>::kOn) {
    static_assert(TeamLds<TP>::kAba <= kTeamRows);
    __shared__ float lds_team[team_lds(TeamLds<TP>::kAba)];
    team_roles<TP>(team_first(), batch, [&](auto W_, const TeamLane& tl) __attribute__((always_inline)) {
      team_aba<TP, EXT, decltype(W_)::value>(tl, tab, SoaIo<TP>{ld}, lds_team, q, qd, tau, fext, ld, qdd);
    });
  }
}

// Inverse dynamics: the way up alone (humanoid 17.5 -> 7.8 us at batch 20001,
// 22.6 -> 12.6 at 65536, 57 -> 44 at 262144, where the 148 MB it reads and writes
// take 29).
template <class TP, bool HAS_QDD, bool EXT, int W, class IO>
RBD_DI void team_rnea(const TeamLane& tl, const float* __restrict__ tab, const IO& io, float* lds_rows, const float* q,
                      const float* qd, const float* qdd, const float* fext, int64_t ld, float* tau) {
  using TM = Team<TP>;
  using ROWS = typename TeamLds<TP>::Id;
  constexpr int NQ = TP::NQ, NV = TP::NV;
  const LdsCol lds{lds_rows + tl.lane};
  const bool owner = TM::may_own(W) && tl.wave == TM::kOwner;
  float qv[NQ], qdv[NV], av[NV];
  team_read<TP, W, true, false>(qv, io, q, tl, owner);
  team_read<TP, W, true, true>(qdv, io, qd, tl, owner);
  if constexpr (HAS_QDD) team_read<TP, W, true, true>(av, io, qdd, tl, owner);
  const RegView qr{qv}, qdr{qdv}, ar{av};
  TeamFd<TP, EXT> s;
  team_id_up<TP, W, ROWS, HAS_QDD>(tab, tab + tl.shift * kBodyStride, qr, qdr, ar,
                                   team_fext<EXT>(fext, ld, tl.shift, tl.b), s, lds.at(team_base<TP, ROWS, W>(tl)),
                                   io.template out<NV>(tau, tl.shift, tl.b));
  if constexpr (TM::may_own(W)) {
    if (owner) team_id_trunk_down<TP, W, HAS_QDD>(tab, qr, qdr, ar, team_fext<EXT>(fext, ld, 0, tl.b), s);
  }
  __syncthreads();
  if constexpr (TM::may_own(W)) {
    if (owner) team_id_trunk<TP, ROWS>(tab, s, lds, io.template out<NV>(tau, 0, tl.b));
  }
}

template <class TP, bool HAS_QDD, bool EXT>
__global__ __launch_bounds__(Team<TP>::kThreads) void k_rnea_team(
    const float* __restrict__ tab, int64_t batch, int64_t ld, const float* __restrict__ q,
    const float* __restrict__ qd, const float* __restrict__ qdd, const float* __restrict__ fext,
    float* __restrict__ tau) {
  if constexpr (Team<TP>::kOn) {
    static_assert(TeamLds<TP>::kId <= kTeamRows);
    __shared__ float lds_team[team_lds(TeamLds<TP>::kId)];
    team_roles<TP>(team_first(), batch, [&](auto W_, const TeamLane& tl) __attribute__((always_inline)) {
      team_rnea<TP, HAS_QDD, EXT, decltype(W_)::value>(tl, tab, SoaIo<TP>{ld}, lds_team, q, qd, qdd, fext, ld, tau);
    });
  }
}

// A wave's view of an output that may be absent, its branches `off` further on.
RBD_DI OutOpt<Out> team_out(float* p, int64_t off, int64_t ld, uint32_t b) {
  return {Out{p ? p + off : nullptr, ld, b}, p != nullptr};
}
template <bool EXT>
RBD_DI auto team_gf(float* p, int64_t ld, int shift, uint32_t b) {
  if constexpr (EXT) return GFOut{{p ? p + 6 * shift * ld : nullptr, ld, b}};
  else return NoGF{};
}

// Forward dynamics' adjoint: the solve with both right-hand sides, after which
// the waves park qdd and lam in LDS (the trunk's are there already), then the
// adjoint sweep, branches first, on fresh views and loading where it uses (held
// in registers, its inputs and qdd and lam spilled 220 B/lane at two waves per
// SIMD). Humanoid: 65.3 -> 25.0 us at batch 64, 74.4 -> 36.0 at 32768, 169 -> 119
// at 131072.
template <class TP, bool EXT, int W, class IO>
RBD_DI void team_fwd_dyn_vjp(const TeamLane& tl, const float* __restrict__ tab, const IO& io, float* lds_rows,
                             const float* q, const float* qd, const float* tau, const float* gqdd, float* gq,
                             float* gqd, float* gtau, const float* fext, float* gfext, int64_t ld) {
  using TM = Team<TP>;
  using ROWS = typename TeamLds<TP>::Fd2;
  using AROWS = typename TeamLds<TP>::template Adj<EXT>;
  constexpr int NQ = TP::NQ, NV = TP::NV, T = TrunkRows<TP>::total();
  const LdsCol lds{lds_rows + tl.lane}, xrow = lds.at(TeamLds<TP>::template vjp_rows<EXT>()), park = lds.at(tl.shift);
  const uint32_t b = tl.b;
  const bool owner = TM::may_own(W) && tl.wave == TM::kOwner;
  {
    float qv[NQ], qdv[NV], tv[NV], gv[NV];
    team_read<TP, W, true, false>(qv, io, q, tl, owner);
    team_read<TP, W, true, true>(qdv, io, qd, tl, owner);
    team_read<TP, W, false, true>(tv, io, tau, tl, owner);
    team_read<TP, W, false, true>(gv, io, gqdd, tl, owner);
    Ltl<TP, 2> F, Ft;
    const RhsTwo<RegView> rhs{RegView{tv}, RegView{gv}};
    const auto gt = io.template opt<NV>(gtau, tl.shift, b), gt_t = io.template opt<NV>(gtau, 0, b);
    team_fd<TP, W, 2, ROWS>(
        tl, owner, tab, RegView{qv}, RegView{qdv}, rhs, rhs, team_fext_opt<EXT>(fext, ld, tl.shift, b),
        team_fext_opt<EXT>(fext, ld, 0, b), lds, xrow, F, Ft,
        [&](int r, int k, float x) __attribute__((always_inline)) {
          park.put(r * NV + k, x);
          if (r == 1) gt(k, x);
        },
        [&](int r, int k, float x) __attribute__((always_inline)) {
          if (r == 1) gt_t(k, x);
        });
  }
  sweep_boundary();
  const IO io2 = io.fresh();
  const int64_t l2 = EXT ? opaque(ld) : ld;
  const float* const t2 = opaque_table(tab);
  const float* const q2 = opaque(q);
  const float* const qd2 = opaque(qd);
  using I = typename IO::I;
  const TeamView<TP, false, I, I> qr{io2.template in<NQ>(q2, tl.shift, b), io2.template in<NQ>(q2, 0, b)};
  const TeamView<TP, true, I, I> qdr{io2.template in<NV>(qd2, tl.shift, b), io2.template in<NV>(qd2, 0, b)};
  const auto solved = [&](int r) __attribute__((always_inline)) {
    auto br = [=](int k) __attribute__((always_inline)) { return park.get(r * NV + k); };
    auto tk = [=](int k) __attribute__((always_inline)) { return xrow.get(r * T + TrunkRows<TP>::row(k)); };
    return TeamView<TP, true, decltype(br), decltype(tk)>{br, tk};
  };
  const auto xr = solved(0), lr = solved(1);
  const LdsCol adj = lds.at(2 * NV);
  AdjState<TP, EXT, EXT> s;
  team_adj_up<TP, W, AROWS>(t2, opaque_table(tab + tl.shift * kBodyStride), s, qr, qdr, xr, lr,
                            io2.template opt<NQ>(gq, tl.shift, b), io2.template opt<NV>(gqd, tl.shift, b),
                            team_fext_opt<EXT>(fext, l2, tl.shift, b), team_gf<EXT>(gfext, l2, tl.shift, b), NoGF{},
                            adj.at(team_base<TP, AROWS, W>(tl)));
  if constexpr (TM::may_own(W)) {
    if (owner)
      team_adj_trunk_down<TP, W>(t2, s, qr, qdr, xr, lr, team_fext_opt<EXT>(fext, l2, 0, b),
                                 team_gf<EXT>(gfext, l2, 0, b));
  }
  __syncthreads();
  if constexpr (TM::may_own(W)) {
    if (owner)
      team_adj_trunk<TP, AROWS>(t2, s, qr, qdr, io2.template opt<NQ>(gq, 0, b), io2.template opt<NV>(gqd, 0, b),
                                NoGF{}, adj);
  }
}

template <class TP, bool EXT>
__global__ __launch_bounds__(Team<TP>::kThreads, EXT ? 1 : 2) void k_fwd_dyn_vjp_team(
    const float* __restrict__ tab, int64_t batch, int64_t ld, const float* __restrict__ q,
    const float* __restrict__ qd, const float* __restrict__ tau, const float* __restrict__ gqdd, float* gq, float* gqd,
    float* gtau, const float* __restrict__ fext, float* gfext) {
  if constexpr (Team<TP>::kOn) {
    static_assert(TeamLds<TP>::template vjp<EXT>() <= kTeamRows);
    __shared__ float lds_team[team_lds(TeamLds<TP>::template vjp<EXT>())];
    team_roles<TP>(team_first(), batch, [&](auto W_, const TeamLane& tl) __attribute__((always_inline)) {
      team_fwd_dyn_vjp<TP, EXT, decltype(W_)::value>(tl, tab, SoaIo<TP>{ld}, lds_team, q, qd, tau, gqdd, gq, gqd,
                                                     gtau, fext, gfext, ld);
    });
  }
}

// Forward dynamics' tangent: the solve for qdd (parked in LDS), the tangent of
// inverse dynamics at it on fresh views, and a second solve with the factor
// that each wave still holds, so M is factored once (humanoid 61.6 -> 23.4 us at
// batch 2048, 68.5 -> 35.5 at 32768, 219 -> 121 at 131072).
template <class TP, bool EXT>
__global__ __launch_bounds__(Team<TP>::kThreads, EXT ? 1 : 2) void k_fwd_dyn_jvp_team(
    const float* __restrict__ tab, int64_t batch, int64_t ld, const float* __restrict__ q,
    const float* __restrict__ qd, const float* __restrict__ tau, const float* __restrict__ dq,
    const float* __restrict__ dqd, const float* __restrict__ dtau, float* qdd, float* dqdd,
    const float* __restrict__ fext, const float* __restrict__ dfext) {
  using TM = Team<TP>;
  if constexpr (TM::kOn) {
    RBD_LANE_IO(TP);
    constexpr int NQ = TP::NQ, NV = TP::NV, T = TrunkRows<TP>::total();
    using ROWS = TeamRows<TP, 16, true, 1>;
    using TROWS = TeamRows<TP, 12, false, 1>;
    // after the first solve its rows hold [qdd | what the tangent hands to the trunk]
    constexpr int kTan = NV + TROWS::total(), kRows = ROWS::total() > kTan ? ROWS::total() : kTan;
    static_assert((kRows + T) <= kTeamRows);
    __shared__ float lds_team[team_lds(kRows + T)];
    team_roles<TP>(team_first(), batch, [&](auto W_, const TeamLane& tl) __attribute__((always_inline)) {
      constexpr int W = decltype(W_)::value;
      const LdsCol lds{lds_team + tl.lane}, xrow = lds.at(kRows), park = lds.at(tl.shift);
      const uint32_t b = tl.b;
      const int64_t off = tl.shift * ld;
      const bool owner = TM::may_own(W) && tl.wave == TM::kOwner;
      Ltl<TP, 1> F, Ft;
      {
        float qv[NQ], qdv[NV], tv[NV];
        team_load<TP, W, true, false>(qv, In{q + off, ld, b}, In{q, ld, b});
        team_load<TP, W, true, true>(qdv, In{qd + off, ld, b}, In{qd, ld, b});
        team_load<TP, W, false, true>(tv, In{tau + off, ld, b}, In{tau, ld, b});
        if constexpr (TM::may_own(W)) {
          if (owner) {
            team_load_trunk<TP, false>(qv, In{q, ld, b});
            team_load_trunk<TP, true>(qdv, In{qd, ld, b});
            team_load_trunk<TP, true>(tv, In{tau, ld, b});
          }
        }
        const RhsOne<RegView> rhs{RegView{tv}};
        team_fd<TP, W, 1, ROWS>(
            tl, owner, tab, RegView{qv}, RegView{qdv}, rhs, rhs, team_fext_opt<EXT>(fext, ld, tl.shift, b),
            team_fext_opt<EXT>(fext, ld, 0, b), lds, xrow, F, Ft,
            [&](int, int k, float x) __attribute__((always_inline)) {
              park.put(k, x);
              if (qdd) Out{qdd + off, ld, b}(k, x);
            },
            [&](int, int k, float x) __attribute__((always_inline)) {
              if (qdd) Out{qdd, ld, b}(k, x);
            });
      }
      sweep_boundary();
      const int64_t l2 = opaque(ld), off2 = tl.shift * l2;
      const float* const t2 = opaque_table(tab);
      const auto qr = team_in<TP, false, In>(opaque(q), off2, l2, b);
      const auto qdr = team_in<TP, true, In>(opaque(qd), off2, l2, b);
      const auto dqr = team_in<TP, false, In>(dq, off2, l2, b);
      const auto dqdr = team_in<TP, true, In>(dqd, off2, l2, b);
      const auto dtr = team_in<TP, true, In>(dtau, off2, l2, b);
      auto xb = [=](int k) __attribute__((always_inline)) { return park.get(k); };
      auto xt = [=](int k) __attribute__((always_inline)) { return xrow.get(TrunkRows<TP>::row(k)); };
      const TeamView<TP, true, decltype(xb), decltype(xt)> xr{xb, xt};
      TanState<TP, EXT> s;
      float rv[NV];  // dtau - d(ID)
      const auto keep = [&](int k, float v) __attribute__((always_inline)) { rv[k] = v; };
      const LdsCol rows = lds.at(NV), c = rows.at(team_base<TP, TROWS, W>(tl));
      const float* const tb2 = opaque_table(tab + tl.shift * kBodyStride);
      team_tan_up<TP, W, TROWS>(t2, tb2, s, qr, qdr, xr, dqr, dqdr, NoFext{}, dtr,
                                team_fext_opt<EXT>(fext, l2, tl.shift, b), team_fext_opt<EXT>(dfext, l2, tl.shift, b),
                                c, keep);
      team_solve_y<TP, W, TROWS>(F, RegView{rv}, c);
      if constexpr (TM::may_own(W)) {
        if (owner)
          team_tan_trunk_down<TP, W>(t2, s, qr, qdr, xr, dqr, dqdr, NoFext{}, team_fext_opt<EXT>(fext, l2, 0, b),
                                     team_fext_opt<EXT>(dfext, l2, 0, b));
      }
      __syncthreads();
      if constexpr (TM::may_own(W)) {
        if (owner) {
          team_tan_trunk<TP, TROWS>(t2, s, dqr, dtr, rows, keep);
          team_solve_trunk<TP, TROWS>(Ft, RegView{rv}, rows, [&](int, int k, float x) __attribute__((always_inline)) {
            xrow.put(TrunkRows<TP>::row(k), x);
            Out{dqdd, l2, b}(k, x);
          });
        }
      }
      __syncthreads();
      team_fd_back<TP, W, 1>(F, [&](int, int k) __attribute__((always_inline)) { return xt(k); },
                             SinkOne<Out>{Out{dqdd + off2, l2, b}});
    });
  }
}

// Poses: every wave walks the trunk above its branches again and writes its
// own bodies, the owner the trunk's (humanoid 16.6 -> 6.0 us at batch 1024, 17.2
// -> 10.0 at 32768; larger batches run one instance per lane).
template <class TP>
__global__ __launch_bounds__(Team<TP>::kThreads) void k_fk_team(const float* __restrict__ tab, int64_t batch,
                                                               int64_t ld, const float* __restrict__ q,
                                                               float* __restrict__ T) {
  using TM = Team<TP>;
  if constexpr (TM::kOn) {
    team_waves<TP>(team_first(), batch, [&](auto W_, const TeamLane& tl) __attribute__((always_inline)) {
      constexpr int W = decltype(W_)::value;
      constexpr bool kOwner = W == TM::kOwner;
      M3 Rw[TP::N];
      V3 pw[TP::N];
      float qv[TP::NQ];
      const In qi{q, ld, tl.b};
      team_load<TP, W, true, false>(qv, qi, qi);
      if constexpr (kOwner) team_load_trunk<TP, false>(qv, qi);
      sfor<0, TP::N>([&](auto I_) __attribute__((always_inline)) {
        constexpr int I = decltype(I_)::value;
        constexpr bool kMine = TM::in(W, I) || (kOwner && TM::trunk(I));
        if constexpr (kMine || TM::above(W, I)) fk_pose<TP, I>(tab, RegView{qv}, Rw, pw);
        if constexpr (kMine) fk_write<TP, I>(tab, Rw, pw, OutNT{T, ld, tl.b});
      });
    });
  }
}

// Jacobians: the frames of a body are written by the wave that has the body
// (humanoid, feet and hands: 45.5 -> 6.2 us at batch 1024).
template <class TP>
__global__ __launch_bounds__(Team<TP>::kThreads) void k_jacobian_team(const float* __restrict__ tab, int64_t batch,
                                                                     int64_t ld, const float* __restrict__ q,
                                                                     JacSlots js, float* __restrict__ J) {
  using TM = Team<TP>;
  if constexpr (TM::kOn) {
    team_waves<TP>(team_first(), batch, [&](auto W_, const TeamLane& tl) __attribute__((always_inline)) {
      constexpr int W = decltype(W_)::value;
      constexpr bool kOwner = W == TM::kOwner;
      M3 Rw[TP::N];
      V3 pw[TP::N];
      float qv[TP::NQ];
      const In qi{q, ld, tl.b};
      team_load<TP, W, true, false>(qv, qi, qi);
      if constexpr (kOwner) team_load_trunk<TP, false>(qv, qi);
      sfor<0, TP::N>([&](auto I_) __attribute__((always_inline)) {
        constexpr int I = decltype(I_)::value;
        constexpr bool kMine = TM::in(W, I) || (kOwner && TM::trunk(I));
        if constexpr (kMine || TM::above(W, I)) fk_pose<TP, I>(tab, RegView{qv}, Rw, pw);
        if constexpr (kMine) jac_frames<TP, I>(Rw, pw, js, J, ld, tl.b);
      });
    });
  }
}

// Mass matrix: the rows of a body are written by the wave that has it; the
// composite inertias of the branches reach the trunk through LDS (humanoid 31.8
// -> 12.0 us at batch 64, 35.6 -> 17.3 at 16384, where the 83 MB it writes take
// 16).
template <class TP>
__global__ __launch_bounds__(Team<TP>::kThreads) void k_crba_team(const float* __restrict__ tab, int64_t batch,
                                                                 int64_t ld, const float* __restrict__ q,
                                                                 float* __restrict__ M) {
  using TM = Team<TP>;
  if constexpr (TM::kOn) {
    constexpr int N = TP::N, NV = TP::NV;
    using ROWS = TeamRows<TP, 10, false, 0>;
    static_assert(ROWS::total() <= kTeamRows);
    __shared__ float lds_team[team_lds(ROWS::total())];
    team_waves<TP>(team_first(), batch, [&](auto W_, const TeamLane& tl) __attribute__((always_inline)) {
      constexpr int W = decltype(W_)::value;
      constexpr bool kOwner = W == TM::kOwner;
      const LdsCol lds{lds_team + tl.lane}, c = lds.at(ROWS::base(W));
      M3 R[N];
      Inr Ic[N];
      float qv[TP::NQ];
      const In qi{q, ld, tl.b};
      team_load<TP, W, true, false>(qv, qi, qi);
      if constexpr (kOwner) team_load_trunk<TP, false>(qv, qi);
      const RegView qr{qv};
      auto put = [&](int r, int k, float v) __attribute__((always_inline)) {
        __builtin_nontemporal_store(v, lane_ptr(M + (int64_t)(r * NV + k) * ld, tl.b));
      };
      auto backward = [&](auto J_) __attribute__((always_inline)) {
        constexpr int J2 = decltype(J_)::value;
        constexpr int P = TP::parent(J2);
        if constexpr (TM::in(W, J2)) {
          crba_write<TP, J2>(tab, R, Ic[J2], put);
          if constexpr (P >= 0) xinr_acc(R[J2], load_r<J2>(tab), Ic[J2], Ic[P]);
        }
      };
      sfor<0, N>([&](auto I_) __attribute__((always_inline)) {
        constexpr int I = decltype(I_)::value;
        if constexpr (TM::in(W, I) || TM::above(W, I) || (kOwner && TM::trunk(I))) {
          if constexpr (!TP::free_body(I)) R[I] = joint_rot<I>(tab, qr(cidx<TP::qofs(I)>));
        }
        if constexpr (TM::attach(W, I)) Ic[I] = Inr{};
        if constexpr (TM::in(W, I)) {
          Ic[I] = load_inr<I>(tab);
          close_subtrees<TP, I, I>(backward);
        }
      });
      sfor<0, N>([&](auto I_) __attribute__((always_inline)) {
        constexpr int I = decltype(I_)::value;
        if constexpr (TM::attach(W, I)) put_inr(c, ROWS::arow(W, I), Ic[I]);
      });
      sfor<0, NV>([&](auto K_) __attribute__((always_inline)) {
        constexpr int K = decltype(K_)::value;
        if constexpr (TM::in(W, TP::body_of(K)) || (kOwner && TM::trunk(TP::body_of(K)))) crba_zeros<TP, K>(put);
      });
      __syncthreads();
      if constexpr (kOwner) {
        sfor<0, N>([&](auto I_) __attribute__((always_inline)) {
          constexpr int I = decltype(I_)::value;
          if constexpr (TM::trunk(I)) Ic[I] = load_inr<I>(tab);
        });
        sfor_rev<0, N>([&](auto J_) __attribute__((always_inline)) {
          constexpr int J2 = decltype(J_)::value;
          constexpr int P = TP::parent(J2);
          if constexpr (TM::trunk(J2)) {
            team_collect<TP, ROWS, J2>(
                lds, [&](const LdsCol& x) __attribute__((always_inline)) { Ic[J2] = Ic[J2] + get_inr(x, 0); });
            crba_write<TP, J2>(tab, R, Ic[J2], put);
            if constexpr (P >= 0) xinr_acc(R[J2], load_r<J2>(tab), Ic[J2], Ic[P]);
          }
        });
      }
    });
  }
}

// Inverse dynamics' tangent and adjoint: one sweep each, as in the middle of
// forward dynamics' (inputs loaded at entry). Adjoint of the humanoid: 33.4 ->
// 12.4 us at batch 64, 38.1 -> 19.9 at 32768.
template <class TP, bool EXT>
__global__ __launch_bounds__(Team<TP>::kThreads) void k_rnea_jvp_team(
    const float* __restrict__ tab, int64_t batch, int64_t ld, const float* __restrict__ q,
    const float* __restrict__ qd, const float* __restrict__ qdd, const float* __restrict__ dq,
    const float* __restrict__ dqd, const float* __restrict__ dqdd, float* __restrict__ dtau,
    const float* __restrict__ fext, const float* __restrict__ dfext) {
  using TM = Team<TP>;
  if constexpr (TM::kOn) {
    RBD_LANE_IO(TP);
    constexpr int NQ = TP::NQ, NV = TP::NV;
    using ROWS = TeamRows<TP, 12, false, 0>;
    static_assert(ROWS::total() <= kTeamRows);
    __shared__ float lds_team[team_lds(ROWS::total())];
    team_roles<TP>(team_first(), batch, [&](auto W_, const TeamLane& tl) __attribute__((always_inline)) {
      constexpr int W = decltype(W_)::value;
      const LdsCol lds{lds_team + tl.lane};
      const uint32_t b = tl.b;
      const int64_t off = tl.shift * ld;
      const bool owner = TM::may_own(W) && tl.wave == TM::kOwner;
      float x[6][NQ];
      const float* const in[6] = {q, dq, qd, qdd, dqd, dqdd};
      sfor<0, 6>([&](auto A_) __attribute__((always_inline)) {
        constexpr int A = decltype(A_)::value;
        team_load<TP, W, true, (A > 1)>(x[A], In{in[A] + off, ld, b}, In{in[A], ld, b});
        if constexpr (TM::may_own(W)) {
          if (owner) team_load_trunk<TP, (A > 1)>(x[A], In{in[A], ld, b});
        }
      });
      const RegView qr{x[0]}, dqr{x[1]}, qdr{x[2]}, ar{x[3]}, dqdr{x[4]};
      const On<RegView> dar{RegView{x[5]}};
      TanState<TP, EXT> s;
      team_tan_up<TP, W, ROWS>(tab, tab + tl.shift * kBodyStride, s, qr, qdr, ar, dqr, dqdr, dar, NoFext{},
                               team_fext_opt<EXT>(fext, ld, tl.shift, b), team_fext_opt<EXT>(dfext, ld, tl.shift, b),
                               lds.at(team_base<TP, ROWS, W>(tl)), Neg<Out>{Out{dtau + off, ld, b}});
      if constexpr (TM::may_own(W)) {
        if (owner)
          team_tan_trunk_down<TP, W>(tab, s, qr, qdr, ar, dqr, dqdr, dar, team_fext_opt<EXT>(fext, ld, 0, b),
                                     team_fext_opt<EXT>(dfext, ld, 0, b));
      }
      __syncthreads();
      if constexpr (TM::may_own(W)) {
        if (owner) team_tan_trunk<TP, ROWS>(tab, s, dqr, NoFext{}, lds, Neg<Out>{Out{dtau, ld, b}});
      }
    });
  }
}

template <class TP, bool EXT>
__global__ __launch_bounds__(Team<TP>::kThreads) void k_rnea_vjp_team(
    const float* __restrict__ tab, int64_t batch, int64_t ld, const float* __restrict__ q,
    const float* __restrict__ qd, const float* __restrict__ qdd, const float* __restrict__ lam,
    float* __restrict__ gq, float* __restrict__ gqd, float* __restrict__ gqdd, const float* __restrict__ fext,
    float* __restrict__ gfext) {
  using TM = Team<TP>;
  if constexpr (TM::kOn) {
    RBD_LANE_IO(TP);
    constexpr int NQ = TP::NQ, NV = TP::NV;
    using ROWS = TeamRows<TP, EXT ? 30 : 18, false, 0>;
    static_assert(ROWS::total() <= kTeamRows);
    __shared__ float lds_team[team_lds(ROWS::total())];
    team_roles<TP>(team_first(), batch, [&](auto W_, const TeamLane& tl) __attribute__((always_inline)) {
      constexpr int W = decltype(W_)::value;
      const LdsCol lds{lds_team + tl.lane};
      const uint32_t b = tl.b;
      const int64_t off = tl.shift * ld;
      const bool owner = TM::may_own(W) && tl.wave == TM::kOwner;
      const float* const t = opaque_table(tab);
      float x[4][NQ];
      const float* const in[4] = {q, qd, qdd, lam};
      sfor<0, 4>([&](auto A_) __attribute__((always_inline)) {
        constexpr int A = decltype(A_)::value;
        team_load<TP, W, true, (A > 0)>(x[A], In{in[A] + off, ld, b}, In{in[A], ld, b});
        if constexpr (TM::may_own(W)) {
          if (owner) team_load_trunk<TP, (A > 0)>(x[A], In{in[A], ld, b});
        }
      });
      const RegView qr{x[0]}, qdr{x[1]}, ar{x[2]}, lr{x[3]};
      const auto neg = [&](float* p, int64_t o) __attribute__((always_inline)) {
        return Neg<OutOpt<Out>>{team_out(p, o, ld, b)};
      };
      const auto gf = [&](int shift) __attribute__((always_inline)) {
        if constexpr (EXT) return Neg<GFOut>{team_gf<EXT>(gfext, ld, shift, b)};
        else return NoGF{};
      };
      AdjState<TP, EXT, EXT> s;
      const float* const tb = opaque_table(tab + tl.shift * kBodyStride);
      team_adj_up<TP, W, ROWS>(t, tb, s, qr, qdr, ar, lr, neg(gq, off), neg(gqd, off),
                               team_fext_opt<EXT>(fext, ld, tl.shift, b), gf(tl.shift),
                               On<OutOpt<Out>>{team_out(gqdd, off, ld, b)}, lds.at(team_base<TP, ROWS, W>(tl)));
      if constexpr (TM::may_own(W)) {
        if (owner)
          team_adj_trunk_down<TP, W>(t, s, qr, qdr, ar, lr, team_fext_opt<EXT>(fext, ld, 0, b), gf(0));
      }
      __syncthreads();
      if constexpr (TM::may_own(W)) {
        if (owner)
          team_adj_trunk<TP, ROWS>(t, s, qr, qdr, neg(gq, 0), neg(gqd, 0), On<OutOpt<Out>>{team_out(gqdd, 0, ld, b)},
                                   lds);
      }
    });
  }
}

// Operational-space control of frame E. One instance per lane: two sweeps
// (bias force with the null-space solve, then the task-space
// solve), the second on fresh views; the torques written by the first are read
// back by the second, so tau is not restrict-qualified. Inputs are loaded
// where they are used (preloading them, as k_fwd_dyn does for large trees,
// held 83 more registers and measured 99 us against 81 us for the humanoid at
// batch 65536 with the sweeps fused).
// A team: branches up, the trunk and the 6x6 task solve by the owner, then J^T z
// on E's branch by the wave that has it; path torques are held back until z is
// known (humanoid, right hand: 65.5 -> 20.1 us at batch 1024, 74.5 -> 45.1 at
// 65536).
template <class TP, int E = TP::N - 1>
__global__ __launch_bounds__(Team<TP>::kOn ? Team<TP>::kThreads : kBlock, Team<TP>::kOn ? 2 : 1) void k_osc(
    const float* __restrict__ tab, int64_t batch, int64_t ld, const float* __restrict__ q,
    const float* __restrict__ qd, const float* __restrict__ tgt, float kp, float kd, float kn, float* tau) {
  using TM = Team<TP>;
  if constexpr (TM::kOn) {
    RBD_LANE_IO(TP);
    constexpr int NQ = TP::NQ, NV = TP::NV;
    using ROWS = TeamRows<TP, 16, true, 1>;
    using EROWS = OscRows<TP, E>;
    using MASK = OscRhs<TP, E>;
    static_assert((ROWS::total() + EROWS::total()) <= kTeamRows);
    __shared__ float lds_team[team_lds(ROWS::total() + EROWS::total())];
    team_waves<TP>(team_first(), batch, [&](auto W_, const TeamLane& tl) __attribute__((always_inline)) {
      constexpr int W = decltype(W_)::value;
      constexpr bool kOwner = W == TM::kOwner, kTask = W == EROWS::kWave;
      const LdsCol lds{lds_team + tl.lane}, ex = lds.at(ROWS::total());
      const uint32_t b = tl.b;
      float qv[NQ], qdv[NV], held[NV];
      const In qi{q, ld, b}, qdi{qd, ld, b}, ti{tgt, ld, b};
      team_load<TP, W, true, false>(qv, qi, qi);
      team_load<TP, W, true, true>(qdv, qdi, qdi);
      if constexpr (kOwner) {
        team_load_trunk<TP, false>(qv, qi);
        team_load_trunk<TP, true>(qdv, qdi);
      }
      const float* const t = opaque_table(tab);
      const RegView qr{qv}, qdr{qdv};
      const Out to{tau, ld, b};
      const auto hold = [&](int k, float v) __attribute__((always_inline)) {
        if (TP::is_anc(TP::body_of(k), E)) held[k] = v;
        else to(k, v);
      };
      struct State : TeamFd<TP, false> {
        V3 p0;
      } s;
      if constexpr (TP::kFree) {
        if constexpr (TM::above(W, 0) || kOwner) s.p0 = {qv[0], qv[1], qv[2]};
      }
      OscHook<TP, E, RegView, In, decltype(hold)> hook{t, qdr, ti, hold, kp, kd, kn};
      hook.init();
      Ltl<TP, kTask ? 7 : 1> F;
      team_fd_up<TP, W, kTask ? 7 : 1, ROWS, MASK>(t, t, qr, qdr, hook, NoFext{}, s, F, lds.at(ROWS::base(W)));
      if constexpr (kTask) {
        sfor<0, NV>([&](auto K_) __attribute__((always_inline)) {
          constexpr int K = decltype(K_)::value;
          if constexpr (TM::above(W, TP::body_of(K)) && TP::is_anc(TP::body_of(K), E)) {
            sfor<0, 6>([&](auto R_) __attribute__((always_inline)) {
              constexpr int r = decltype(R_)::value;
              ex.put(cidx<EROWS::yrow(K)> + r, team_yshare<TP, W, K, r + 1, MASK>(F));
            });
          }
        });
        int n = EROWS::kG;
#pragma unroll
        for (int i = 0; i < 6; ++i) {
#pragma unroll
          for (int j = 0; j <= i; ++j) ex.put(n++, hook.G[i][j]);
          ex.put(EROWS::kA + i, hook.a[i]);
        }
        if constexpr (EROWS::anchor() >= 0) {
#pragma unroll
          for (int i = 0; i < 9; ++i) ex.put(EROWS::kT + i, hook.A.a[i]);
          ex.put(EROWS::kT + 9, hook.o.x); ex.put(EROWS::kT + 10, hook.o.y); ex.put(EROWS::kT + 11, hook.o.z);
        }
      }
      if constexpr (kOwner) {
        // the trunk's motion (its hook starts afresh: a wave may own both E and the trunk)
        team_fd_trunk_down<TP, W>(t, qr, qdr, NoFext{}, s);
      }
      __syncthreads();
      float z[6];
      if constexpr (kOwner) {
        OscHook<TP, E, RegView, In, decltype(hold)> top{t, qdr, ti, hold, kp, kd, kn};
        top.init();
        if constexpr (EROWS::kWave >= 0) {
          int n = EROWS::kG;
#pragma unroll
          for (int i = 0; i < 6; ++i) {
#pragma unroll
            for (int j = 0; j <= i; ++j) top.G[i][j] = ex.get(n++);
            top.a[i] = ex.get(EROWS::kA + i);
          }
          if constexpr (EROWS::anchor() >= 0) {
#pragma unroll
            for (int i = 0; i < 9; ++i) top.A.a[i] = ex.get(EROWS::kT + i);
            top.o = {ex.get(EROWS::kT + 9), ex.get(EROWS::kT + 10), ex.get(EROWS::kT + 11)};
          }
        } else {
          sfor<0, E + 1>([&](auto I_) __attribute__((always_inline)) {
            if constexpr (TP::is_anc(decltype(I_)::value, E)) top.motion(I_, s);
          });
        }
        Ltl<TP, 7> Ft;
        team_fd_trunk<TP, 7, ROWS, MASK>(t, OscTrunkHook<TP, E, decltype(top)>{top, ex}, s, lds, Ft);
        chol6_solve(top.G, top.a, z);
        if constexpr (EROWS::kWave >= 0) {
#pragma unroll
          for (int i = 0; i < 6; ++i) lds.put(i, z[i]);
        }
        sfor<0, NV>([&](auto K_) __attribute__((always_inline)) {
          constexpr int K = decltype(K_)::value;
          if constexpr (TM::trunk(TP::body_of(K)) && TP::is_anc(TP::body_of(K), E))
            to(K, held[K] + top.task_torque(K, z));
        });
      }
      __syncthreads();
      if constexpr (kTask) {
#pragma unroll
        for (int i = 0; i < 6; ++i) z[i] = lds.get(i);
        sfor<0, NV>([&](auto K_) __attribute__((always_inline)) {
          constexpr int K = decltype(K_)::value;
          if constexpr (TM::in(W, TP::body_of(K)) && TP::is_anc(TP::body_of(K), E))
            to(K, held[K] + hook.task_torque(K, z));
        });
      }
    });
  } else {
    RBD_LANE_IO(TP);
    const uint32_t b = lane_id();
    if (b >= batch) return;
    float ypath[TP::NV], astar[6];
    osc_sweep_bias<TP, E>(tab, In{q, ld, b}, In{qd, ld, b}, In{tgt, ld, b}, kp, kd, kn, OutAlias{tau, ld, b}, ypath,
                          astar);
    sweep_boundary();
    // the second sweep on fresh views (see k_fwd_dyn_vjp)
    const int64_t l2 = opaque(ld);
    osc_sweep_task<TP, E>(opaque_table(tab), In{opaque(q), l2, b}, ypath, astar, OutAlias{tau, l2, b},
                          InAlias{tau, l2, b});
  }
}

// ---- packed launch for the serving runtime. One launch serves many requests
// of one (model, operation): the work is cut into tiles of 64 instances (one
// wave), every tile belongs to one request, and a fixed grid of waves strides
// over the tiles, so the same launch (and a graph that captured it) serves any
// number of requests. A tree that is shared out over a team gives every tile to
// a block, any other to a wave (at every size: a group that is large enough for
// one instance per lane to be better takes longer to copy than to compute). Request arrays are instance-major, exactly as the client
// handed them over: coordinate c of instance i at p[i * n + c].
template <class TP, int OP>
struct PackedShape {  // threads of a block and waves per SIMD to leave registers for
  static constexpr int kThreads = Team<TP>::kOn ? Team<TP>::kThreads : kBlock;
  static constexpr int kOcc = !Team<TP>::kOn ? 1 : (OP == kOpFwdDyn ? 3 : 2);
};
template <class TP, int OP>
__global__ __launch_bounds__((PackedShape<TP, OP>::kThreads), (PackedShape<TP, OP>::kOcc)) void k_packed(
    const float* __restrict__ tab, const uint8_t* __restrict__ table) {
  const PackedHdr* hdr = reinterpret_cast<const PackedHdr*>(table);
  const int32_t* tile_req = reinterpret_cast<const int32_t*>(table + sizeof(PackedHdr));
  const PackedReq* reqs = reinterpret_cast<const PackedReq*>(table + hdr->req_offset);
  const int n_tiles = hdr->n_tiles;
  if constexpr (Team<TP>::kOn) {
    // a team per tile, the same code as the direct calls
    using L = TeamLds<TP>;
    constexpr int kRows = OP == kOpFwdDyn ? L::kAba : (OP == kOpRnea ? L::kId : L::template vjp<false>());
    static_assert(kRows <= kTeamRows);
    __shared__ float lds_team[team_lds(kRows)];
    for (int t = blockIdx.x; t < n_tiles; t += gridDim.x) {
      const PackedReq& R = reqs[__builtin_amdgcn_readfirstlane(tile_req[t])];
      const float* const q = R.in[0];
      const float* const qd = R.in[1];
      const float* const x2 = R.in[2];
      const RowIo io{};
      team_roles<TP>((t - R.first_tile) * kTileLanes, R.batch,
                     [&](auto W_, const TeamLane& tl) __attribute__((always_inline)) {
        constexpr int W = decltype(W_)::value;
        if constexpr (OP == kOpFwdDyn)
          team_aba<TP, false, W>(tl, tab, io, lds_team, q, qd, x2, nullptr, 0, R.out[0]);
        else if constexpr (OP == kOpRnea)
          team_rnea<TP, true, false, W>(tl, tab, io, lds_team, q, qd, x2, nullptr, 0, R.out[0]);
        else
          team_fwd_dyn_vjp<TP, false, W>(tl, tab, io, lds_team, q, qd, x2, R.in[3], R.out[0], R.out[1], R.out[2],
                                         nullptr, nullptr, 0);
      });
      __syncthreads();  // the next tile reuses the rows
    }
  } else {
    const int lane = threadIdx.x & (kTileLanes - 1);
    const int wave = (int)((blockIdx.x * (int64_t)blockDim.x + threadIdx.x) / kTileLanes);
    const int n_waves = (int)(((int64_t)gridDim.x * blockDim.x) / kTileLanes);
    constexpr int NQ = TP::NQ, NV = TP::NV;
    for (int t = wave; t < n_tiles; t += n_waves) {
      const int r = __builtin_amdgcn_readfirstlane(tile_req[t]);
      const PackedReq& R = reqs[r];
      const int64_t i = (int64_t)(t - R.first_tile) * kTileLanes + lane;
      if (i >= R.batch) continue;
      const InRow q{R.in[0] + i * NQ}, qd{R.in[1] + i * NV}, x2{R.in[2] + i * NV};
      if constexpr (OP == kOpFwdDyn) {
        fwd_dyn_lane<TP, 1>(tab, q, qd, RhsOne<InRow>{x2}, SinkOne<OutRow>{OutRow{R.out[0] + i * NV}});
      } else if constexpr (OP == kOpRnea) {
        rnea_lane<TP, true>(tab, q, qd, x2, OutRow{R.out[0] + i * NV});
      } else {
        float* gqd = R.out[1] + i * NV;
        float* gtau = R.out[2] + i * NV;
        if constexpr (NV > 16) {
          // the two sweeps on fresh views, as in k_fwd_dyn_vjp
          fwd_dyn_lane<TP, 2>(tab, q, qd, RhsTwo<InRow>{x2, InRow{R.in[3] + i * NV}},
                              SinkTwo<RowAlias>{RowAlias{gqd}, RowAlias{gtau}});
          sweep_boundary();
          id_adjoint_lane<TP>(opaque_table(tab), InRow{opaque(R.in[0]) + i * NQ}, InRow{opaque(R.in[1]) + i * NV},
                              RowAlias::In{gqd}, RowAlias::In{gtau}, OutRow{R.out[0] + i * NQ}, RowAlias{gqd});
        } else {
          vjp_lane_parked<TP>(tab, q, qd, x2, InRow{R.in[3] + i * NV}, OutRow{R.out[0] + i * NQ}, RowAlias{gqd},
                              RowAlias{gtau}, RowAlias::In{gqd}, RowAlias::In{gtau});
        }
      }
    }
  }
}

}  // namespace rbd
