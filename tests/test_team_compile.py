"""Run-time compilation of the adjoint of inverse dynamics of a team for trees whose moved tables the
compiler keeps in vector registers: each in a process of its own, which a failing compilation used to end."""
from __future__ import annotations

import os
import re
import subprocess
import sys

import pytest

from paper_2604_04310_amd import build as B

KERNELS = re.findall(r"X\((KID_\w+),", open(os.path.join(B.CSRC, "rbd_kernel_ids.hpp")).read())


@pytest.mark.parametrize("kernel", ["KID_RNEA_VJP_TEAM", "KID_RNEA_VJP_EXT_TEAM"])
@pytest.mark.parametrize("floating,parent", [
    (True, [-1, 0, 1, 2, 0, 4, 4, 4, 7, 8, 9, 10, 0, 12, 13]),
    (False, [-1, 0, 1, 2, 3, 4, 5, 6, 7, 8, 6, 0, 11, 0, 13, 14, 0, 16])])
def test_moved_tables_compile(tmp_path, floating, parent, kernel):
    code = ("import paper_2604_04310_amd as rbd\n"
            f"rbd.precompile_topology({parent}, {floating}, {str(tmp_path)!r}, kernel={KERNELS.index(kernel)})\n")
    r = subprocess.run([sys.executable, "-c", code], cwd=os.path.dirname(B.PKG), capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-500:]
    assert len([f for f in os.listdir(tmp_path) if f.endswith(".hsaco")]) == 1
