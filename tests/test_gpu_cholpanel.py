"""GPU tests of the periodizer's QR with Cholesky panels: against the column
steps over panel remainders and row remainders, and where a panel's columns
are too nearly dependent for it."""
from __future__ import annotations

import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def mfs():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    import paper_1506_05083_amd as m
    m.lib()
    return m


def rel(x, y):
    return float(np.linalg.norm(x - y) / np.linalg.norm(y))


@pytest.mark.parametrize("lat,nb", [
    (dict(p=14, N0=3.0, M1=6), 16),      # 144 rows: one part-filled chunk; halves of 126 and 111 columns
    (dict(p=14, N0=3.0, M1=6), 64),
    (dict(p=15, N0=2.2, M1=6), 32),      # 140 columns on 144 rows: the last panels have few rows left
    (dict(p=24, N0=10, M1=20), 64),      # 1600 rows, several chunks
    (dict(p=1, N0=2.2, M1=2), 16),       # 16 rows, fewer columns than a panel
    (dict(p=10, N0=1.5, M1=4), 16),      # rank 121 of 125: dependent columns, back to column steps
    (dict(p=30, N0=3.0, M1=16), 64),     # harmonics far past what the walls resolve: nearly dependent panels
])
def test_cholesky_panels_match_column_steps(mfs, monkeypatch, lat, nb):
    """Same kept ranks, amplitudes and fields within 1e-9: both are backward
    stable factorisations of the same equilibrated Q, and a one-ulp change of Q
    moves the most sensitive of these amplitudes (rank 121 of 125) by 3e-12;
    the factorisations are allowed a few hundred ulps."""
    pr = W.small_periodic(nwaves=3)
    b, la = pr.body, W.with_(pr.lattice, **lat)
    sh = b.shape
    ctx = mfs.create(0)
    op = mfs.build_operator(ctx, [mfs.BodySpec(b.M, b.N, b.P, b.q, b.k,
                                               mfs.polar_geometry(sh.a, sh.eps, sh.j, b.M, b.N, b.tau, b.colloc))])
    op.factor_modes(1e-10)
    L = mfs.lattice(la.ex, la.ey, la.z0, la.p, la.N0, la.M1)
    monkeypatch.setenv("MFS_QR_NB", str(nb))
    got = {}
    for panel in ("chol", "steps"):
        monkeypatch.setenv("MFS_QR_PANEL", panel)
        got[panel] = mfs.solve_incident(ctx, op, L, [(w.theta, w.phi) for w in pr.waves], tol=1e-12, maxit=100,
                                        targets=pr.targets, q_field=pr.q_field)
    for r, s in zip(got["chol"], got["steps"]):
        e = max(rel(r.a, s.a), rel(r.b, s.b), rel(r.field, s.field))
        print(f"[chol {lat} nb={nb}] rank {r.q_rank} {s.q_rank} of {r.nq_cols}, {e:.1e}", flush=True)
        assert r.q_rank == s.q_rank and e < 1e-9
