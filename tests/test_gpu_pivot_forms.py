"""GPU test of which pivoted QR a triangle takes: one launch with a workgroup a
matrix up to 128 columns, a launch pair a column up to 255, sketched pivots from
256 on."""
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


@pytest.mark.parametrize("N,form", [(64, "one"), (65, "one"), (127, "one"), (128, "one"), (129, "unblocked"),
                                    (130, "unblocked"), (200, "unblocked"), (255, "unblocked"), (256, "sketched")])
def test_default_form(mfs, monkeypatch, N, form):
    """The default has the bits of its form, and not those of the others; the forms'
    singular values agree to N eps of the largest (each is backward stable)."""
    b = W.small_periodic().body
    ctx = mfs.create(0)
    monkeypatch.setenv("MFS_QR_NB", "64")
    kv = np.array([[0.3, 0.2, -1.0]])
    got = {}
    for f in ("default", "one", "unblocked", "sketched"):
        if f == "default":
            monkeypatch.delenv("MFS_QRCP", raising=False)
        elif f == "one" and N > 128:
            continue
        else:
            monkeypatch.setenv("MFS_QRCP", f)
        op = mfs.build_operator(ctx, [mfs.BodySpec(N + 9, N, 4, 64, b.k, mfs.polar_geometry(
            b.shape.a, b.shape.eps, b.shape.j, N + 9, N, b.tau, b.colloc))])
        op.factor_modes(1e-10)
        got[f] = op.singular_values(0), mfs.apply_solution_op(op, mfs.rhs_modes(op, kv)).cpu().numpy()
    for f, (sv, c) in got.items():
        if f == "default":
            continue
        same = bool((sv == got["default"][0]).all() and (c == got["default"][1]).all())
        assert same == (f == form), f
        assert np.max(np.abs(sv - got["default"][0])) <= N * np.finfo(float).eps * sv.max()
