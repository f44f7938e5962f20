"""GPU test that the periodizer's Cholesky panels are what factors Q, and that the
halves they cannot factor, alone or among others, go back to column steps."""
from __future__ import annotations

import os
import re
import subprocess
import sys

import pytest

pytestmark = pytest.mark.gpu

# in a process of its own: the library looks for MFS_PROGRESS once
CHILD = """
import numpy as np
import paper_1506_05083_amd as mfs
import workloads as W
pr = W.small_periodic(nwaves=3)
b, sh = pr.body, pr.body.shape
ctx = mfs.create(0)
op = mfs.build_operator(ctx, [mfs.BodySpec(b.M, b.N, b.P, b.q, b.k,
                                           mfs.polar_geometry(sh.a, sh.eps, sh.j, b.M, b.N, b.tau, b.colloc))])
op.factor_modes(1e-10)
for lat in (dict(p=14, N0=3.0, M1=6), dict(p=15, N0=2.2, M1=6), dict(p=24, N0=10, M1=20), dict(p=1, N0=2.2, M1=2),
            dict(p=30, N0=3.0, M1=16), dict(p=10, N0=1.5, M1=4)):
    la = W.with_(pr.lattice, **lat)
    L = mfs.lattice(la.ex, la.ey, la.z0, la.p, la.N0, la.M1)
    for ws in ([0, 1, 2], [0], [1], [2]):
        mfs.solve_incident(ctx, op, L, [(pr.waves[i].theta, pr.waves[i].phi) for i in ws], tol=1e-9, maxit=60,
                           targets=pr.targets, q_field=pr.q_field)
"""


def test_halves_factored_by_cholesky_panels():
    """None again by column steps where the columns are independent; on the lattice
    whose Q has rank 121 of 125 some halves and not all, the same ones with other
    waves and alone."""
    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    env = dict(os.environ, MFS_PROGRESS="1", PYTHONPATH=root)
    for v in ("MFS_QR_PANEL", "MFS_QR_NB"):
        env.pop(v, None)
    r = subprocess.run([sys.executable, "-c", CHILD], env=env, cwd=root, capture_output=True, text=True, timeout=100)
    assert r.returncode == 0, r.stderr[-2000:]
    got = [(int(a), int(n)) for a, n in re.findall(r"(\d+) of (\d+) halves again by column steps", r.stderr)]
    assert len(got) == 24, r.stderr
    for i in range(5):
        assert got[4 * i: 4 * i + 4] == [(0, 6), (0, 2), (0, 2), (0, 2)], i
    both, alone = got[20], got[21:]
    assert 0 < both[0] < 6 and sum(a for a, _ in alone) == both[0], got[20:]
