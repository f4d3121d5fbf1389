"""The C entry points of the team kernels with a leading dimension above the batch: NaN in the inputs'
padding is never read, the outputs' padding stays untouched, and every result equals the contiguous call's
bit for bit (the same kernel on the same values). Operational-space control at the edges of a block of 64
instances, with the frame on the owner's branch, on another wave's, and in the trunk."""
from __future__ import annotations

import ctypes as C

import numpy as np
import pytest

import oracle as O
import workloads as W
from oracle import controllers as CT
from paper_2604_04310_amd.build import PREBUILT
from tests._helpers import targets_near
from tests.test_gpu_controllers import KD, KN, KP, floor_osc, within_bar

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

TREES = {"humanoid30": (True, W.humanoid().parent), "quadruped13f": PREBUILT["quadruped13f"],
         "arms25": PREBUILT["arms25"]}
SENTINEL = -77.25


@pytest.fixture(scope="module")
def rbd():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2604_04310_amd as rbd
    rbd.lib()
    return rbd


def desc_of(name, seed):
    floating, par = TREES[name]
    return W.random_tree(list(par), floating, seed, rotated=True, gravity=W.tilted_gravity(seed + 1))


@pytest.mark.parametrize("batch", [1, 65, 200])
@pytest.mark.parametrize("name", list(TREES))
def test_rows_apart(rbd, name, batch):
    desc = desc_of(name, 840)
    m = rbd.Model(desc, 0)
    nq, nv, nb, ld = desc.nq, desc.nv, desc.n_bodies, batch + 3
    st = W.states(desc, batch, 842 + batch)
    rng = np.random.Generator(np.random.PCG64(843))
    f32 = lambda x: torch.tensor(np.ascontiguousarray(np.asarray(x).reshape(batch, -1).T),  # noqa: E731
                                 dtype=torch.float32, device="cuda")
    draw = lambda rows: f32(rng.normal(size=(batch, rows)))  # noqa: E731
    q, qd, tau, w, x = f32(st.q), f32(st.qd), f32(st.tau), draw(nv), draw(nv)
    dq, dqd, dx, fx, dfx = draw(nq), draw(nv), draw(nv), draw(6 * nb), draw(6 * nb)
    tgt = f32(targets_near(O.fk(desc, st.q)[:, nb - 1], 844))
    frames = np.arange(0, nb, 2, dtype=np.int32)
    fp, nf = frames.ctypes.data_as(C.POINTER(C.c_int32)), len(frames)
    L, stream = rbd.lib(), torch.cuda.current_stream().cuda_stream

    def both(fn, args, out_rows):
        """The C function with ld = batch, then ld = batch + 3; args: tensors, None, or plain values as given,
        "out" for an output."""
        got = []
        for wide in (batch, ld):
            keep, call, outs, rows = [], [], [], iter(out_rows)
            for a in args:
                if isinstance(a, torch.Tensor):
                    buf = torch.full((a.shape[0], wide), float("nan"), device="cuda")
                    buf[:, :batch] = a
                    keep.append(buf)
                    call.append(buf.data_ptr())
                elif isinstance(a, str):
                    outs.append(torch.full((next(rows), wide), SENTINEL, device="cuda"))
                    call.append(outs[-1].data_ptr())
                else:
                    call.append(a)
            assert fn(m.handle, batch, wide, *call, stream) == 0, L.rbd_last_error()
            torch.cuda.synchronize()
            got.append([o.cpu() for o in outs])
        for a, b in zip(*got):
            assert torch.isfinite(a).all() and torch.equal(a, b[:, :batch])
            assert (b[:, batch:] == SENTINEL).all(), "a column past the batch was written"

    o = "out"
    both(L.rbd_fk, [q, o], [12 * nb])
    both(L.rbd_jacobian, [q, nf, fp, o], [6 * nv * nf])
    both(L.rbd_crba, [q, o], [nv * nv])
    for f, df in ((None, None), (fx, dfx)):
        both(L.rbd_fwd_dyn, [q, qd, tau, f, o], [nv])
        both(L.rbd_aba, [q, qd, tau, f, o], [nv])
        both(L.rbd_rnea, [q, qd, w, f, o], [nv])
        both(L.rbd_rnea, [q, qd, None, f, o], [nv])
        both(L.rbd_rnea_jvp, [q, qd, w, f, dq, dqd, dx, df, o], [nv])
        both(L.rbd_fwd_dyn_jvp, [q, qd, tau, f, dq, dqd, dx, df, o, o], [nv, nv])
        gf, rows = (o, [nq, nv, nv, 6 * nb]) if f is not None else (None, [nq, nv, nv])
        both(L.rbd_rnea_vjp, [q, qd, w, f, x, o, o, o, gf], rows)
        both(L.rbd_fwd_dyn_vjp, [q, qd, tau, f, x, o, o, o, gf], rows)
    both(L.rbd_osc, [q, qd, nb - 1, tgt, KP, KD, KN, o], [nv])


@pytest.mark.parametrize("batch", [1, 63, 64, 65])
@pytest.mark.parametrize("name,frame", [("humanoid30", f) for f in (0, 6, 15, 22, 29)]
                         + [("quadruped13f", f) for f in (3, 12)])
def test_osc_blocks(rbd, name, frame, batch):
    desc = desc_of(name, 850)
    m = rbd.Model(desc, 0)
    st = W.states(desc, batch, 851 + frame)
    tgt = W._f32(targets_near(O.fk(desc, st.q)[:, frame], 852 + frame))
    gpu = lambda x: torch.tensor(np.ascontiguousarray(x.reshape(batch, -1).T), dtype=torch.float32,  # noqa: E731
                                 device="cuda")
    tau = rbd.osc(m, gpu(st.q), gpu(st.qd), gpu(tgt), KP, KD, KN, frame=frame)
    torch.cuda.synchronize()
    ref = CT.osc(desc, st.q, st.qd, frame, tgt, KP, KD, KN)
    assert within_bar(tau.double().cpu().numpy().T, ref, floor_osc(desc, st.q, frame, ref)) < 1.0
