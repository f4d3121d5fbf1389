"""Trees with several roots that are shared out over a team of waves: where every branch hangs on the
world, the waves hand nothing over. Every kernel of such a tree compiles (on the CPU: instantiated for
gfx950 by the compiler's front end), and the served and packed operations and operational-space control
agree with the oracle (the direct calls run in the tests over all installed trees)."""
from __future__ import annotations

import os
import shutil
import subprocess
from concurrent.futures import ThreadPoolExecutor

import numpy as np
import pytest

import oracle as O
import workloads as W
from oracle import controllers as CT
from paper_2604_04310_amd import build as B
from tests._helpers import rel_err, targets_near, vjp_err

ROOTS = {name: B.PREBUILT[name] for name in ("arms18", "arms25", "arms18f")}
COMPILED = {**ROOTS, "chains20": (False, [-1, *range(9), -1, *range(10, 19)]),
            "arms28": (False, [x + 7 * k if x >= 0 else -1 for k in range(4) for x in range(-1, 6)]),
            "joints17": (False, [-1] * 17), "joints20f": (True, [-1] * 15)}

KERNELS = r"""
#include <hip/hip_runtime.h>
#include "rbd_kernel_ids.hpp"
#include "rbd_kernels.hpp"
namespace rbd {
using TP = Tree<TREE>;
#define RBD_ADDRESS(id, part, ...) (const void*)&__VA_ARGS__,
const void* const kernels[] = {RBD_KERNELS(RBD_ADDRESS)};
template <int... E>
struct Osc {
  const void* const at[sizeof...(E)] = {(const void*)&k_osc<TP, E>...};
};
const Osc<FRAMES> osc;
}
"""


def test_every_kernel_compiles(tmp_path):
    if not (os.path.exists(B.HIPCC) or shutil.which(B.HIPCC)):
        pytest.skip("no hipcc")
    src = tmp_path / "kernels.hip"
    src.write_text(KERNELS)

    def compile_tree(item):
        name, (floating, par) = item
        frames = sorted({0, len(par) // 2, len(par) - 1})
        r = subprocess.run([B.HIPCC, "--offload-arch=gfx950", "-std=c++17", "--cuda-device-only", "-fsyntax-only",
                            f"-I{B.CSRC}", f"-DTREE={'true' if floating else 'false'},{','.join(map(str, par))}",
                            f"-DFRAMES={','.join(map(str, frames))}", str(src)], capture_output=True, text=True)
        return name, r.returncode, [x for x in r.stderr.splitlines() if "error" in x]

    with ThreadPoolExecutor(4) as ex:
        results = list(ex.map(compile_tree, COMPILED.items()))
    assert [(n, rc, e) for n, rc, e in results if rc or e] == []


@pytest.fixture(scope="module")
def rbd():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2604_04310_amd as rbd
    rbd.lib()
    return rbd


def desc_of(name):
    floating, par = ROOTS[name]
    return W.random_tree(par, floating, 860, rotated=True, gravity=W.tilted_gravity(861))


@pytest.mark.gpu
@pytest.mark.parametrize("name", list(ROOTS))
def test_served_and_packed(rbd, name):
    """Requests of 1, 64 and 131 instances: the server (graphs of all three operations) and the packed call."""
    import torch
    desc = desc_of(name)
    m = rbd.Model(desc, 0)
    cases = []
    for k, batch in enumerate((1, 64, 131)):
        st = W.states(desc, batch, 862 + k)
        g = W._f32(W.cotangent(desc.nv, batch, 870 + k))
        cases += [(rbd.OP_FWD_DYN, [st.q, st.qd, st.tau], [O.fwd_dyn(desc, st.q, st.qd, st.tau)]),
                  (rbd.OP_RNEA, [st.q, st.qd, g], [O.rnea(desc, st.q, st.qd, g)]),
                  (rbd.OP_FWD_DYN_VJP, [st.q, st.qd, st.tau, g],
                   list(O.fwd_dyn_vjp_fd(desc, st.q, st.qd, st.tau, g)))]

    def check(op, got, ref):
        if op == rbd.OP_FWD_DYN_VJP:
            assert vjp_err(got, ref) < 1e-3
        else:
            assert rel_err(got[0], ref[0]) < 1e-4

    srv = rbd.Server(arena_bytes=64 << 20, n_streams=2)
    tickets = [srv.submit(m, op, [np.ascontiguousarray(x, dtype=np.float32) for x in ins]) for op, ins, _ in cases]
    for (op, _, ref), (t, outs) in zip(cases, tickets):
        assert srv.wait(t, 60.0) == 0
        check(op, [o.astype(np.float64) for o in outs], ref)
    srv.close()
    for op in (rbd.OP_FWD_DYN, rbd.OP_RNEA, rbd.OP_FWD_DYN_VJP):
        reqs = [([torch.from_numpy(np.ascontiguousarray(x, dtype=np.float32)).cuda() for x in ins],
                 [torch.full((len(ins[0]), r), float("nan"), device="cuda") for r in rbd.op_shapes(m, op)[1]])
                for o, ins, _ in cases if o == op]
        rbd.packed_static(m, op, reqs)
        torch.cuda.synchronize()
        for (_, outs), ref in zip(reqs, [r for o, _, r in cases if o == op]):
            check(op, [x.double().cpu().numpy() for x in outs], ref)


def check_osc(rbd, desc, frame, batch):
    import torch
    from tests.test_gpu_controllers import KD, KN, KP, floor_osc, within_bar
    m = rbd.Model(desc, 0)
    st = W.states(desc, batch, 880 + frame)
    tgt = W._f32(targets_near(O.fk(desc, st.q)[:, frame], 881 + frame))
    gpu = lambda x: torch.tensor(np.ascontiguousarray(x.reshape(batch, -1).T), dtype=torch.float32,  # noqa: E731
                                 device="cuda")
    tau = rbd.osc(m, gpu(st.q), gpu(st.qd), gpu(tgt), KP, KD, KN, frame=frame)
    torch.cuda.synchronize()
    ref = CT.osc(desc, st.q, st.qd, frame, tgt, KP, KD, KN)
    assert within_bar(tau.double().cpu().numpy().T, ref, floor_osc(desc, st.q, frame, ref)) < 1.0


@pytest.mark.gpu
def test_osc_beside_a_free_body(rbd):
    """A small tree (one instance per lane): the frame's root stands beside the free base."""
    check_osc(rbd, W.random_tree([-1, -1, 1, 2, 3, 4, 5], True, 865, rotated=True), 6, 65)


@pytest.mark.gpu
@pytest.mark.parametrize("batch", [1, 65])
@pytest.mark.parametrize("name,frame", [("arms18", 5), ("arms18", 17), ("arms25", 6), ("arms25", 24),
                                        ("arms18f", 0), ("arms18f", 6), ("arms18f", 12)])
def test_osc(rbd, name, frame, batch):
    """Frames at the end of an arm and on a free body that carries nothing."""
    check_osc(rbd, desc_of(name), frame, batch)
