"""GPU tests of the neighbour sum's forms: one to sixteen right-hand sides (vector
and matrix-core sums), mirror-paired surfaces and walls and user targets, at
source and target counts off the tiles, each right-hand side against its own
sum."""
from __future__ import annotations

import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def body():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    import paper_1506_05083_amd as mfs
    b = W.small_periodic().body
    ctx = mfs.create(0)
    op = mfs.build_operator(ctx, [mfs.BodySpec(b.M, b.N - 1, b.P, b.q, b.k, mfs.polar_geometry(
        b.shape.a, b.shape.eps, b.shape.j, b.M, b.N - 1, b.tau, b.colloc))])
    return mfs, ctx, b, op


@pytest.mark.parametrize("nrhs", [1, 2, 3, 4, 5, 6, 7, 8, 9, 12, 13, 16])
@pytest.mark.parametrize("which", ["surface", "walls", "user", "user_deriv"])
def test_right_hand_sides_match_their_own_sums(body, which, nrhs):
    """The largest difference from the one-wave sum, 1e-13 of the largest value:
    both add the same S terms (under 2^10 a slice) in another order, each with a
    kernel value a few ulps of 1 + k R off."""
    import torch
    mfs, _, b, op = body
    rng = np.random.default_rng(nrhs)
    sig = torch.tensor(rng.standard_normal((nrhs, b.P, b.N - 1)) + 1j * rng.standard_normal((nrhs, b.P, b.N - 1))).cuda()
    ab = np.exp(2j * np.pi * rng.random((nrhs, 2)))
    L = mfs.lattice(1.0, 1.0, 0.8, 10, 3.0, 10)
    kw = {}
    if which.startswith("user"):
        t = rng.standard_normal((131, 6)) * 0.2 + np.array([0, 0, 2.0, 0, 0, 0])
        kw = dict(user=t, want=int(which == "user_deriv"))
        ts = mfs.TARGETS_USER
    else:
        ts = mfs.TARGETS_SURFACE if which == "surface" else mfs.TARGETS_WALLS
    got = mfs.neighbour_sum(op, L, sig, ab, ts, **kw).cpu().numpy()
    for r in range(nrhs):
        one = mfs.neighbour_sum(op, L, sig[r:r + 1].contiguous(), ab[r:r + 1], ts, **kw).cpu().numpy()[0]
        assert np.max(np.abs(got[r] - one)) < 1e-13 * np.max(np.abs(one)), r


@pytest.mark.parametrize("kr", [1e-3, 1.0, 50.0, 1e3, 1e5, 2e9, 4e14, 3e15])
def test_kernel_phase_over_distances(body, kr):
    """One unit source strength at growing distances against the formula on the
    CPU: the magnitude to 1e-14, the phase to the rounding of k R (4 eps k R) up to
    the distance where that is the whole circle."""
    import torch
    mfs, ctx, b, op = body
    sig = torch.zeros((1, b.P, b.N - 1), dtype=torch.complex128)
    sig[0, 0, 0] = 1.0
    R = kr / b.k
    g = mfs.polar_geometry(b.shape.a, b.shape.eps, b.shape.j, b.M, b.N - 1, b.tau, b.colloc)
    y = np.array([g["srho"][0], 0.0, g["sz"][0]])
    d = np.array([0.6, 0.0, 0.8])
    x = y + R * d
    c = torch.zeros((1, b.P, b.N - 1), dtype=torch.complex128)
    c[0, :, 0] = 1.0 / b.P     # the node l = 0 alone: sum over modes
    u = mfs.field_free(op, c.cuda(), b.P, x[None]).cpu().numpy()[0, 0]
    s = mfs.point_strengths(op, c.cuda(), b.P).cpu().numpy()[0]
    ph = 2 * np.pi * np.arange(b.P) / b.P
    src = np.stack([g["srho"][0] * np.cos(ph), g["srho"][0] * np.sin(ph), np.full(b.P, g["sz"][0])], -1)
    r = np.linalg.norm(x - src, axis=1)
    ref = np.sum(np.exp(1j * b.k * r) / (4 * np.pi * r) * s[:, 0])
    mag = np.sum(np.abs(s[:, 0]) / (4 * np.pi * r))
    assert np.isfinite(u)
    tol = 1e-14 + 4 * np.finfo(float).eps * kr * (1 + np.linalg.norm(x) / R)
    assert abs(u - ref) < min(tol, 2.0) * mag + 1e-14 * mag
