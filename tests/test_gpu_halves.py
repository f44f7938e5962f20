"""GPU test of the periodizer's two halves (Q split by the cell's mirror
symmetry in z) where they go wrong most easily: a half with more columns than
wall rows, so that it carries zero rows and loses rank, and a truncation whose
scale is the larger half's."""
from __future__ import annotations

import numpy as np
import pytest

import workloads as W
from oracle import geometry, onebody, periodic

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("p,N0,M1", [(10, 1.5, 4), (14, 3.0, 6), (1, 2.2, 2)])
def test_halves_against_oracle(p, N0, M1):
    """Ranks equal to the unsplit oracle SVD's, amplitudes and fields within
    1e-9 of it.  (10, 1.5, 4): 125 columns on 128 rows, the even half 68 on
    64, rank 121; a one-ulp change of Q moves these amplitudes by 3e-12, and
    the blocked factorisations are allowed a few hundred ulps."""
    import torch
    assert torch.cuda.is_available()
    import paper_1506_05083_amd as mfs
    pr = W.small_periodic(nwaves=2)
    b, lat = pr.body, W.with_(pr.lattice, p=p, N0=N0, M1=M1)
    g = geometry.build_geometry(b)
    ps = periodic.PeriodicSolver(b, lat, g, onebody.modal_blocks(b, g))
    sh = b.shape
    ctx = mfs.create(0)
    op = mfs.build_operator(ctx, [mfs.BodySpec(b.M, b.N, b.P, b.q, b.k,
                                               mfs.polar_geometry(sh.a, sh.eps, sh.j, b.M, b.N, b.tau, b.colloc))])
    op.factor_modes(1e-10)
    L = mfs.lattice(lat.ex, lat.ey, lat.z0, lat.p, lat.N0, lat.M1)
    res = mfs.solve_incident(ctx, op, L, [(w.theta, w.phi) for w in pr.waves], tol=1e-12, maxit=100,
                             targets=pr.targets, q_field=pr.q_field)
    for w, r in zip(pr.waves, res):
        ps.set_wave(w)
        o = ps.solve(onebody.rhs_modes(b, g, w), tol=1e-12)
        u, _ = ps.field_and_grad(o["c"], o["d"], pr.targets, pr.q_field, want_grad=False)
        assert np.array_equal(r.m, ps.orders.m) and np.array_equal(r.n, ps.orders.n)
        assert r.nq_cols == ps.Q.shape[1] and r.q_rank == ps.Qf[1].size
        for x, y in ((r.a, o["a"]), (r.b, o["b"]), (r.field, u)):
            err = np.linalg.norm(x - y) / np.linalg.norm(y)
            print(f"[halves p={p}] {err:.1e}", flush=True)
            assert err < 1e-9
