"""GPU tests of what a periodic solve takes its near field from by default."""
from __future__ import annotations

import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu

EXPANSIONS, STORED = 4, 1


@pytest.fixture(scope="module")
def mfs():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    import paper_1506_05083_amd as m
    m.lib()
    return m


def problem(mfs, a=0.3, **body):
    pr = W.small_periodic()
    b = W.with_(pr.body, shape=W.Shape(a, 0.1, 3), **body)
    ctx = mfs.create(0)
    op = mfs.build_operator(ctx, [mfs.BodySpec(b.M, b.N, b.P, b.q, b.k, mfs.polar_geometry(
        a, 0.1, 3, b.M, b.N, b.tau, b.colloc))])
    op.factor_modes(1e-10)
    la = pr.lattice
    L = mfs.lattice(la.ex, la.ey, la.z0, la.p, la.N0, la.M1)
    waves = [(w.theta, w.phi) for w in W.sample_waves(b.k, la, 16, seed=5, theta_max=1.3)]

    def solve(ws):
        res, tm = mfs.solve_incident(ctx, op, L, ws, tol=1e-13, maxit=100, targets=pr.targets, q_field=64,
                                     timing=True, allow_notconv=True)
        return res, int(tm["near_mode"])
    return op, waves, solve


def rel(x, y):
    return float(np.linalg.norm(x - y) / np.linalg.norm(y))


def same(r, s):
    """Both forms agree to rounding: the expansions are cut at 1e-15 of a source's
    field, the residuals are 1e-13, and the problems amplify by under a hundred."""
    return max(rel(r.a, s.a), rel(r.b, s.b), rel(r.field, s.field)) < 1e-11


@pytest.mark.parametrize("kw,nw,mode", [
    (dict(), 2, EXPANSIONS),                       # 255 MB stored, 59 MB a wave
    (dict(), 4, EXPANSIONS),
    (dict(), 8, STORED),
    (dict(), 16, STORED),
    (dict(a=0.22), 16, EXPANSIONS),                # 23 MB a wave
    (dict(N=60, M=72, P=28), 16, EXPANSIONS),      # half a surface of 1008 targets: no mirror pairs, two launches
    (dict(N=48, M=64, P=24), 12, STORED),
])
def test_waves_against_stored_values(mfs, monkeypatch, kw, nw, mode):
    monkeypatch.delenv("MFS_NEAR_EXPANSION", raising=False)
    _, waves, solve = problem(mfs, **kw)
    res, got = solve(waves[:nw])
    assert got == mode
    one, got = solve(waves[:1])
    assert got == EXPANSIONS and same(res[0], one[0])


def test_budget_for_one_waves_matrices(mfs, monkeypatch):
    """A budget that holds one wave's matrices but not three waves' (nor all stored
    values): the sums change their form with the number of waves, the results stay
    the same to rounding."""
    monkeypatch.delenv("MFS_NEAR_EXPANSION", raising=False)
    op, waves, solve = problem(mfs)
    op.set_near_field_budget(140 << 20)
    one, got = solve(waves[:1])
    assert got == EXPANSIONS
    res, got = solve(waves[:3])
    assert got not in (EXPANSIONS, STORED)
    assert same(res[0], one[0])
