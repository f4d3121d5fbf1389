"""Kernels that share a tree out over a team of waves (rbd_team.hpp), at the edges of their blocks
of 64 instances, in arrays with a leading dimension above the batch whose padding must stay
untouched; trees whose branches are copies of each other, are not, and hang on several trunk bodies."""
from __future__ import annotations

import numpy as np
import pytest

import oracle as O
import workloads as W
from paper_2604_04310_amd.build import PREBUILT
from tests._helpers import rel_err
from tests._models import TREE12

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

TOL = 1e-4  # the bar of the parity tests of forward dynamics
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
