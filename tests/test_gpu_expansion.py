"""GPU tests of the near field by spherical-wave expansions: solves forced
onto it (MFS_NEAR_EXPANSION=2) against the same solves on point sums
(MFS_NEAR_EXPANSION=0) over the sizes at which its kernels change course, and
against the CPU oracle."""
from __future__ import annotations

import numpy as np
import pytest

import workloads as W
from oracle import geometry, onebody, periodic

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def mfs():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    import paper_1506_05083_amd as m
    m.lib()
    return m


def problem(kind, **lat):
    if kind == "cup":
        pr = W.small_periodic_cup(nwaves=9)
    elif kind == "penetrable":
        pr = W.small_periodic_transmission(nwaves=9)
    else:
        pr = W.small_periodic(nwaves=9)
    body = pr.body if kind != "few_angles" else W.with_(pr.body, P=12)
    la = W.with_(pr.lattice, **lat)
    waves = tuple(W.sample_waves(body.k, la, 9, seed=21, theta_max=1.3))
    return W.with_(pr, body=body, lattice=la, waves=waves)


def operator(mfs, ctx, pr):
    b, sh = pr.body, pr.body.shape
    g = (mfs.transmission_geometry if pr.km > 0 else mfs.body_geometry)(sh, b.M, b.N, b.tau, b.colloc)
    op = mfs.build_operator(ctx, [mfs.BodySpec(b.M, b.N, b.P, b.q, b.k, g, pr.km)])
    op.factor_modes(1e-10)
    return op


def rel(x, y):
    return float(np.linalg.norm(x - y) / np.linalg.norm(y))


@pytest.mark.parametrize("kind,lat,nw", [
    ("polar", {}, 1),                                # two waves a group, one of them padding
    ("polar", dict(ex=1.1, ey=1.25, p=8), 3),        # rectangular lattice; harmonics below the target degree
    ("polar", dict(p=50, M1=26), 2),                 # harmonics above the target degree
    ("polar", dict(M1=2, p=1, N0=2.2), 9),           # one node a wall half-row; more than eight waves
    ("few_angles", {}, 5),                           # several azimuthal orders to a mode bin
    ("cup", {}, 2),
    ("penetrable", {}, 3),                           # value and derivative rows, interior coefficients skipped
])
def test_expansion_matches_point_sums(mfs, monkeypatch, kind, lat, nw):
    """Amplitudes and fields of both forms agree to 1e-11: the expansions are
    cut at 1e-15 of a source's field, the GMRES residual is 1e-13, and these
    discretisations amplify either by less than a thousand."""
    pr = problem(kind, **lat)
    ctx = mfs.create(0)
    op = operator(mfs, ctx, pr)
    la = pr.lattice
    L = mfs.lattice(la.ex, la.ey, la.z0, la.p, la.N0, la.M1)
    got = {}
    for mode, near in (("2", 4), ("0", 1)):
        monkeypatch.setenv("MFS_NEAR_EXPANSION", mode)
        res, tm = mfs.solve_incident(ctx, op, L, [(w.theta, w.phi) for w in pr.waves[:nw]], tol=1e-13, maxit=100,
                                     targets=pr.targets, q_field=pr.q_field, timing=True, allow_notconv=True)
        assert int(tm["near_mode"]) == near
        got[mode] = res
    for i, (r, s) in enumerate(zip(got["2"], got["0"])):
        ea, eb, eu = rel(r.a, s.a), rel(r.b, s.b), rel(r.field, s.field)
        print(f"[expansion {kind} {lat}] wave {i} iters {r.iters} {s.iters} a {ea:.1e} b {eb:.1e} u {eu:.1e}", flush=True)
        assert max(ea, eb, eu) < 1e-11


def test_expansion_against_oracle(mfs, monkeypatch):
    """Two waves of the small periodic body against the oracle to 1e-10, as
    the point sums are."""
    monkeypatch.setenv("MFS_NEAR_EXPANSION", "2")
    pr = W.small_periodic(nwaves=2)
    b, la = pr.body, pr.lattice
    ctx = mfs.create(0)
    op = operator(mfs, ctx, pr)
    L = mfs.lattice(la.ex, la.ey, la.z0, la.p, la.N0, la.M1)
    res = mfs.solve_incident(ctx, op, L, [(w.theta, w.phi) for w in pr.waves], tol=1e-12, maxit=100,
                             targets=pr.targets, q_field=pr.q_field)
    g = geometry.build_geometry(b)
    ps = periodic.PeriodicSolver(b, la, g, onebody.modal_blocks(b, g))
    for w, r in zip(pr.waves, res):
        ps.set_wave(w)
        o = ps.solve(onebody.rhs_modes(b, g, w), tol=1e-12)
        u, _ = ps.field_and_grad(o["c"], o["d"], pr.targets, pr.q_field, want_grad=False)
        assert max(rel(r.a, o["a"]), rel(r.b, o["b"]), rel(r.field, u)) < 1e-10


def test_wide_bodies_keep_point_sums(mfs, monkeypatch):
    """A body whose bounding sphere nearly fills the cell has no short
    expansion: the solve keeps the stored values even when asked for it."""
    monkeypatch.setenv("MFS_NEAR_EXPANSION", "2")
    pr = problem("polar")
    pr = W.with_(pr, body=W.with_(pr.body, shape=W.Shape(0.42, 0.1, 3)))
    ctx = mfs.create(0)
    op = operator(mfs, ctx, pr)
    la = pr.lattice
    L = mfs.lattice(la.ex, la.ey, la.z0, la.p, la.N0, la.M1)
    _, tm = mfs.solve_incident(ctx, op, L, [(pr.waves[0].theta, pr.waves[0].phi)], tol=1e-8, maxit=60, timing=True,
                               allow_notconv=True)
    assert int(tm["near_mode"]) == 1


def test_server_on_expansions(mfs, monkeypatch):
    """Waves entering and leaving the server's slots with per-slot expansion
    matrices give the plain solves' results."""
    monkeypatch.setenv("MFS_NEAR_EXPANSION", "2")
    pr = problem("polar")
    ctx = mfs.create(0)
    op = operator(mfs, ctx, pr)
    la = pr.lattice
    L = mfs.lattice(la.ex, la.ey, la.z0, la.p, la.N0, la.M1)
    waves = [(w.theta, w.phi) for w in pr.waves]
    ref = [mfs.solve_incident(ctx, op, L, [w], tol=1e-12, maxit=100, targets=pr.targets, q_field=pr.q_field)[0]
           for w in waves]
    srv = mfs.Server(ctx, op, L, slots=3, admit_batch=2, tol=1e-12, maxit=100, targets=pr.targets,
                     q_field=pr.q_field, hbm_budget=48 << 30)
    try:
        got = [srv.wait(t)[0] for t in [srv.submit(*w) for w in waves]]
    finally:
        srv.close()
    for r, s in zip(got, ref):
        assert max(rel(r.a, s.a), rel(r.b, s.b), rel(r.field, s.field)) < 1e-11
