"""GPU test of the inverse of a QR'd matrix's triangle at the edges of its 16-
and 64-column blocks, through the full-rank pseudoinverse that is built on it."""
from __future__ import annotations

import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M,N", [(2, 1), (18, 15), (20, 16), (20, 17), (40, 33), (64, 48), (70, 63), (72, 64), (73, 65),
                                 (90, 81), (140, 128), (150, 129), (230, 193)])
def test_pseudoinverse_at_block_edges(M, N):
    """A c of the coefficients c = V S^+ U^H f against the projection of f on the
    kept range.  V S^+ is the triangle's inverse times U: each of its N-term sums is
    rounded relative to its terms, so A c is off by N eps times the kept part's
    condition, more where the cutoff falls between close singular values (the
    kept range turns by that much); ten of that."""
    import torch
    import paper_1506_05083_amd as mfs
    b = W.small_periodic().body
    ctx = mfs.create(0)
    op = mfs.build_operator(ctx, [mfs.BodySpec(M, N, 4, 64, b.k, mfs.polar_geometry(
        b.shape.a, b.shape.eps, b.shape.j, M, N, b.tau, b.colloc))])
    A = op.blocks().cpu().numpy().transpose(0, 2, 1)
    op.factor_modes(1e-10)
    rng = np.random.default_rng(M)
    f = rng.standard_normal((4, M)) + 1j * rng.standard_normal((4, M))
    c = mfs.apply_solution_op(op, torch.tensor(f[None]).cuda()).cpu().numpy()[0]
    # modes 0, 1, 2, -1: the block of |n|
    for i, n in enumerate((0, 1, 2, 1)):
        u, s, _ = np.linalg.svd(A[n], full_matrices=False)
        k = int(np.sum(s > 1e-10 * s[0]))
        u = u[:, :k]
        gap = s[k - 1] - (s[k] if k < N else 0.0)
        e = float(np.linalg.norm(A[n] @ c[i] - u @ (u.conj().T @ f[i])) / np.linalg.norm(f[i]))
        tol = 10 * N * np.finfo(float).eps * s[0] / gap
        print(f"[trinv {M} x {N}] mode {i}: kept {k}, {e:.1e} of {tol:.1e}", flush=True)
        assert e < tol
