"""GPU tests of the pivoted QR of the triangles at the edges of its forms: one
workgroup a matrix up to 256 columns, sketched above, with the sketch's pivots
in one launch up to 1536 remaining columns; and of the QR's one-launch panels
at row counts around whole waves."""
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


@pytest.mark.parametrize("M,N", [
    (2, 1), (4, 3), (33, 32), (34, 33), (65, 64), (66, 65), (127, 100), (128, 128), (129, 127), (193, 192),
    (257, 255), (256, 256), (300, 257), (512, 500), (513, 513), (1040, 1030), (1560, 1540),
])
def test_singular_values_at_edges(mfs, M, N):
    """Singular values of the GPU's own blocks against LAPACK, 1e-13 of the
    largest or N eps where that is larger (each side is backward stable), and the
    kept ranks within one of LAPACK's count."""
    b = W.small_periodic().body
    ctx = mfs.create(0)
    op = mfs.build_operator(ctx, [mfs.BodySpec(M, N, 2, 64, b.k, mfs.polar_geometry(
        b.shape.a, b.shape.eps, b.shape.j, M, N, b.tau, b.colloc))])
    blocks = op.blocks().cpu().numpy().transpose(0, 2, 1)
    ranks = op.factor_modes(1e-10)
    sv = op.singular_values(0)
    tol = max(1e-13, N * np.finfo(float).eps)
    for n in range(blocks.shape[0]):
        s = np.linalg.svd(blocks[n], compute_uv=False)
        e = float(np.max(np.abs(sv[n][: s.size] - s)) / s[0])
        print(f"[pivots {M} x {N}] mode {n}: rank {ranks[n]}, singular values {e:.1e}", flush=True)
        assert abs(int(ranks[n]) - int(np.sum(s > 1e-10 * s[0]))) <= 1
        assert e < tol


@pytest.mark.parametrize("M,N,P", [(48, 40, 4), (36, 17, 4), (210, 200, 16), (620, 600, 4)])
def test_jacobi_rounds_in_one_launch_match_three(mfs, monkeypatch, M, N, P):
    """A round of the blocked Jacobi in one launch and in three: the same kept
    ranks, singular values within 1e-13 of the largest or N eps (both converge
    to the same relative orthogonality)."""
    b = W.small_periodic().body
    ctx = mfs.create(0)
    got = []
    for form in ("1", "0"):
        monkeypatch.setenv("MFS_JAC_ROUND", form)
        op = mfs.build_operator(ctx, [mfs.BodySpec(M, N, P, 64, b.k, mfs.polar_geometry(
            b.shape.a, b.shape.eps, b.shape.j, M, N, b.tau, b.colloc))])
        got.append((np.array(op.factor_modes(1e-10)), op.singular_values(0)))
    (r1, s1), (r3, s3) = got
    e = max(float(np.max(np.abs(a - c)) / c[0]) for a, c in zip(s1, s3))
    print(f"[jacobi rounds {M} x {N}] {e:.1e}", flush=True)
    assert (r1 == r3).all() and e < max(1e-13, N * np.finfo(float).eps)


def test_jacobi_streams_give_the_same_bits(mfs, monkeypatch):
    """Matrices of three bodies' modes in one group or in four, each group's
    rounds on its own stream: every matrix runs its own rounds, so the singular
    values and ranks are the same bits."""
    b = W.small_periodic().body
    ctx = mfs.create(0)
    specs = [mfs.BodySpec(M, N, P, 64, b.k, mfs.polar_geometry(b.shape.a, b.shape.eps, b.shape.j, M, N, b.tau, b.colloc))
             for M, N, P in ((48, 40, 16), (120, 100, 8), (36, 17, 4))]
    got = []
    for ns in ("1", "4"):
        monkeypatch.setenv("MFS_JAC_STREAMS", ns)
        op = mfs.build_operator(ctx, specs)
        got.append((np.array(op.factor_modes(1e-10)), [op.singular_values(i) for i in range(3)]))
    (r1, s1), (r4, s4) = got
    assert (r1 == r4).all()
    for x, y in zip(s1, s4):
        assert all((np.asarray(u) == np.asarray(v)).all() for u, v in zip(x, y))
