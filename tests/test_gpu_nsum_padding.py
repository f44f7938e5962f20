"""GPU test of the neighbour sum's last chunks of sources: the slots past the last
source hold no point of their own, so no target is singular but the sources."""
from __future__ import annotations

import numpy as np
import pytest

import workloads as W
from oracle import geometry, kernel, periodic

pytestmark = pytest.mark.gpu


def tolerance(b, r):
    return 8 * np.finfo(float).eps * (b.k * r + b.P * b.N)


@pytest.fixture(scope="module")
def body():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    import paper_1506_05083_amd as mfs
    b = W.small_periodic().body
    b = W.with_(b, N=b.N - 1)
    s = b.shape
    op = mfs.build_operator(mfs.create(0), [mfs.BodySpec(
        b.M, b.N, b.P, b.q, b.k, mfs.polar_geometry(s.a, s.eps, s.j, b.M, b.N, b.tau, b.colloc))])
    return mfs, b, op, geometry.source_ring_points(geometry.build_geometry(b), b.P).reshape(-1, 3)


@pytest.mark.parametrize("nrhs", [1, 3, 6, 7, 16])
@pytest.mark.parametrize("z", [1e3, -1e3, 999.5])
def test_targets_far_on_the_axes_of_the_images(body, nrhs, z):
    """Targets on the axis of the body and of its images, values and derivatives,
    against the closed formula: a phase is off by the rounding of k R on either side,
    and a sum of S terms by S eps of their magnitudes."""
    import torch
    mfs, b, op, y = body
    rng = np.random.default_rng(3)
    sig = rng.standard_normal((nrhs, b.P, b.N)) + 1j * rng.standard_normal((nrhs, b.P, b.N))
    ab = np.exp(2j * np.pi * rng.random((nrhs, 2)))
    lat = W.with_(W.small_periodic().lattice, ex=1.1, ey=1.25)
    L = mfs.lattice(lat.ex, lat.ey, lat.z0, lat.p, lat.N0, lat.M1)
    x = np.array([[a * lat.ex, c * lat.ey, z] for a in (-1, 0, 1) for c in (-1, 0, 1)])
    for want, n in ((0, [0.0, 0.0, 0.0]), (1, [0.6, 0.0, 0.8])):
        t = np.hstack([x, np.tile(n, (len(x), 1))])
        got = mfs.neighbour_sum(op, L, torch.from_numpy(sig).cuda(), ab, mfs.TARGETS_USER, user=t,
                                want=want).cpu().numpy()
        for r in range(nrhs):
            ref, mag = 0.0, 0.0
            for _, w, shift in periodic.image_list(lat, ab[r, 0], ab[r, 1], periodic.NEAR9):
                d = (x[:, None, :], y[None, :, :] + shift)
                K = kernel.dG_dnx(b.k, d[0], np.array(n), d[1]) if want else kernel.G(b.k, *d)
                ref = ref + w * (K @ sig[r].reshape(-1))
                mag = mag + np.abs(K) @ np.abs(sig[r].reshape(-1))
            assert np.max(np.abs(got[r] - ref) / mag) < tolerance(b, 1e3), (want, r)


@pytest.mark.parametrize("nrhs", [1, 7])
def test_free_field_far_on_the_axis(body, nrhs):
    """The same for the free-space field at (0, 0, 1000)."""
    import torch
    mfs, b, op, y = body
    rng = np.random.default_rng(4)
    c = torch.from_numpy(rng.standard_normal((nrhs, b.P, b.N)) + 1j * rng.standard_normal((nrhs, b.P, b.N))).cuda()
    s = mfs.point_strengths(op, c, b.P).cpu().numpy().reshape(nrhs, -1)
    x = np.array([[0.0, 0.0, 1e3], [0.0, 0.0, 2.0]])
    K = kernel.G(b.k, x[:, None, :], y[None, :, :])
    got = mfs.field_free(op, c, b.P, x).cpu().numpy()
    assert np.max(np.abs(got - s @ K.T) / (np.abs(s) @ np.abs(K).T)) < tolerance(b, 1e3)
