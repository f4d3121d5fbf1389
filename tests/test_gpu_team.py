"""Kernels that share a tree out over a team of waves (rbd_team.hpp), at the edges of their blocks
of 64 instances, in arrays with a leading dimension above the batch whose padding must stay
untouched; trees whose branches are copies of each other, are not, and hang on several trunk bodies."""
from __future__ import annotations

import numpy as np
import pytest

import oracle as O
import workloads as W
from paper_2604_04310_amd.build import PREBUILT
from tests._helpers import rel_err, vjp_err
from tests._models import TREE12

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

TOL = 1e-4  # the bar of the parity tests of forward dynamics
# ... and those of the other operations
TOL_TAU, TOL_M, TOL_KIN, TOL_VJP = 1e-4, 1e-5, 1e-5, 1e-3
TREES = {"tree12f": (True, TREE12), "humanoid30": (True, W.humanoid().parent), **PREBUILT}
SENTINEL = -77.25


@pytest.fixture(scope="module")
def rbd():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2604_04310_amd as rbd
    rbd.lib()
    return rbd


def padded(x, ld):
    """Host [B, rows] as a [rows, B] view of a [rows, ld] array; NaN in the padding."""
    x = x.reshape(len(x), -1).T
    buf = torch.full((x.shape[0], ld), float("nan"), dtype=torch.float32, device="cuda")
    buf[:, :x.shape[1]] = torch.tensor(np.ascontiguousarray(x), dtype=torch.float32, device="cuda")
    return buf[:, :x.shape[1]]


def outputs(rows, batch, ld):
    buf = torch.full((rows, ld), SENTINEL, dtype=torch.float32, device="cuda")
    return buf, buf[:, :batch]


def result(buf, batch):
    torch.cuda.synchronize()
    x = buf.double().cpu().numpy()
    assert (x[:, batch:] == SENTINEL).all(), "a column past the batch was written"
    return x[:, :batch].T


@pytest.mark.parametrize("batch", [1, 63, 64, 65, 200])
@pytest.mark.parametrize("name", list(TREES))
def test_fwd_dyn_blocks(rbd, name, batch):
    fl, par = TREES[name]
    desc = W.random_tree(par, fl, 810, rotated=True, gravity=W.tilted_gravity(811))
    m = rbd.Model(desc, 0)
    st = W.states(desc, batch, 812 + batch)
    rng = np.random.Generator(np.random.PCG64(813))
    fext = W._f32(rng.normal(0.0, 5.0, size=(batch, desc.n_bodies, 6)))
    ld = batch + 3
    args = [padded(x, ld) for x in (st.q, st.qd, st.tau)]
    for fx in (None, fext):
        buf, out = outputs(desc.nv, batch, ld)
        rbd.fwd_dyn(m, *args, out=out, fext=None if fx is None else padded(fx, ld))
        assert rel_err(result(buf, batch), O.fwd_dyn(desc, st.q, st.qd, st.tau, fext=fx)) < TOL


def check_all(rbd, m, desc, batch, seed, ops, sample=None):
    """The operations in ops on one batch; the oracle on the instances of sample (all if None)."""
    st = W.states(desc, batch, seed)
    rng = np.random.Generator(np.random.PCG64(seed + 1))
    norm = lambda rows, sd=1.0: W._f32(rng.normal(0.0, sd, size=(batch, rows)))  # noqa: E731
    nq, nv, nb = desc.nq, desc.nv, desc.n_bodies
    qdd, x, dq, dqd, dx = norm(nv), norm(nv), norm(nq), norm(nv), norm(nv)
    fext, dfext = norm(6 * nb, 5.0), norm(6 * nb)
    idx = np.arange(batch) if sample is None else np.asarray(sample)
    P = lambda a: padded(a, batch)  # noqa: E731
    S = lambda a: np.ascontiguousarray(a[idx])  # noqa: E731

    def got(t):
        torch.cuda.synchronize()
        assert t.shape[1] == batch and bool(torch.isfinite(t).all())
        return t[:, torch.as_tensor(idx, device="cuda")].double().cpu().numpy().T

    q, qd, tau = P(st.q), P(st.qd), P(st.tau)
    qs, qds, taus, ws = S(st.q), S(st.qd), S(st.tau), S(qdd)
    forces = [(None, None, None, None), (P(fext), S(fext), P(dfext), S(dfext))]
    if "fd" in ops:
        for f, fs, _, _ in forces:
            ref = O.fwd_dyn(desc, qs, qds, taus, fext=fs)
            for fn in (rbd.fwd_dyn, rbd.aba):
                assert rel_err(got(fn(m, q, qd, tau, fext=f)), ref) < TOL
    if "rnea" in ops:
        for f, fs, _, _ in forces:
            for w, wo in ((P(qdd), ws), (None, None)):
                assert rel_err(got(rbd.rnea(m, q, qd, w, fext=f)), O.rnea(desc, qs, qds, wo, fext=fs)) < TOL_TAU
    if "crba" in ops:
        assert rel_err(got(rbd.crba(m, q)), O.crba(desc, qs)) < TOL_M
    if "fk" in ops:
        assert rel_err(got(rbd.fk(m, q)), O.fk(desc, qs)) < TOL_KIN
    if "jacobian" in ops:  # every body, and three of them twice
        frames = np.concatenate([np.arange(nb), np.arange(0, nb, max(1, nb // 2))]).astype(np.int32)
        J = got(rbd.jacobian(m, q, frames))
        ref = O.jacobian(desc, qs, frames).reshape(len(idx), -1)
        assert rel_err(J, ref) < TOL_KIN and np.all(J[ref == 0.0] == 0.0)
    if "vjp" in ops:
        for f, fs, _, _ in forces:
            out = rbd.fwd_dyn_vjp(m, q, qd, tau, P(x), fext=f, want_fext=f is not None)
            ref = O.fwd_dyn_vjp_fd(desc, qs, qds, taus, S(x), fext=fs)
            assert vjp_err([got(o) for o in out], list(ref)) < TOL_VJP
    if "rnea_vjp" in ops:
        for f, fs, _, _ in forces:
            out = rbd.rnea_vjp(m, q, qd, P(qdd), P(x), fext=f, want_fext=f is not None)
            ref = O.rnea_vjp_fd(desc, qs, qds, ws, S(x), fext=fs, want_fext=f is not None)
            assert vjp_err([got(o) for o in out], list(ref)) < TOL_VJP
    t, ts = [P(a) for a in (dq, dqd, dx)], [S(a) for a in (dq, dqd, dx)]
    if "jvp" in ops:
        for f, fs, df, dfs in forces:
            d = got(rbd.fwd_dyn_jvp(m, q, qd, tau, *t, fext=f, dfext=df))
            ref = O.fwd_dyn_jvp_fd(desc, qs, qds, taus, *ts, fext=fs, dfext=dfs)
            assert vjp_err([d], [ref]) < TOL_VJP
    if "rnea_jvp" in ops:
        for f, fs, df, dfs in forces:
            d = got(rbd.rnea_jvp(m, q, qd, P(qdd), *t, fext=f, dfext=df))
            ref = O.rnea_jvp_fd(desc, qs, qds, ws, *ts, fext=fs, dfext=dfs)
            assert vjp_err([d], [ref]) < TOL_VJP


OPS = ("fd", "rnea", "crba", "fk", "jacobian", "vjp", "rnea_vjp", "jvp", "rnea_jvp")


@pytest.mark.parametrize("batch", [1, 65])
@pytest.mark.parametrize("name", list(TREES))
def test_every_operation_blocks(rbd, name, batch):
    fl, par = TREES[name]
    desc = W.random_tree(par, fl, 820, rotated=True, gravity=W.tilted_gravity(821))
    check_all(rbd, rbd.Model(desc, 0), desc, batch, 822 + batch, OPS)


@pytest.mark.parametrize("name,batch,ops", [
    (n, b, (op,)) for n in ("humanoid30", "quadruped13f")
    for op, limit in (("jacobian", 32768), ("crba", 40960), ("fk", 57344)) for b in (limit, limit + 1)] + [
    ("quadruped13f", b, ("fd", "rnea", "vjp", "rnea_vjp", "jvp", "rnea_jvp")) for b in (81920, 81921)])
def test_both_sides_of_the_batch_limits(rbd, name, batch, ops):
    """Team and one-instance-per-lane kernels on either side of the batch where one takes over."""
    fl, par = TREES[name]
    desc = W.random_tree(par, fl, 830, rotated=True, gravity=W.tilted_gravity(831))
    sample = [0, 1, 63, 64, 127, batch // 2, batch - 66, batch - 65, batch - 2, batch - 1]
    check_all(rbd, rbd.Model(desc, 0), desc, batch, 832, ops, sample)
