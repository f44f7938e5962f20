"""GPU tests of the device memory cache's small blocks: reuse across calls and
streams, the statistics, and giving everything back."""
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


def test_small_blocks_are_reused_without_changing_results(mfs):
    """Many short calls in a row, on the default and on a side stream, whose
    temporaries are released while the next call's work is queued: every result
    has the bits of the first."""
    import torch
    b = W.small_periodic().body
    sh = b.shape
    ctx = mfs.create(0)
    op = mfs.build_operator(ctx, [mfs.BodySpec(b.M, b.N, b.P, b.q, b.k,
                                               mfs.polar_geometry(sh.a, sh.eps, sh.j, b.M, b.N, b.tau, b.colloc))])
    op.factor_modes(1e-10)
    kv = np.array([[0.3, 0.2, -1.0], [0.1, -0.4, -1.0]])
    tg = W.fibonacci_sphere(70, 2.0)
    side = torch.cuda.Stream()
    first = None
    for i in range(40):
        with torch.cuda.stream(side if i % 3 == 2 else torch.cuda.current_stream()):
            c = mfs.apply_solution_op(op, mfs.rhs_modes(op, kv))
            u = mfs.field_free(op, c, b.P, tg).cpu().numpy()
        torch.cuda.synchronize()
        first = u if first is None else first
        assert (u == first).all()


def test_released_memory_is_given_back(mfs):
    """After an operator is gone its bytes are no longer in use but cached, and
    release_cached_memory leaves nothing cached."""
    b = W.small_periodic().body
    sh = b.shape
    ctx = mfs.create(0)
    base = mfs.memory_stats(0)["in_use"]
    op = mfs.build_operator(ctx, [mfs.BodySpec(b.M, b.N, b.P, b.q, b.k,
                                               mfs.polar_geometry(sh.a, sh.eps, sh.j, b.M, b.N, b.tau, b.colloc))])
    op.factor_modes(1e-10)
    assert mfs.memory_stats(0)["in_use"] > base
    del op
    st = mfs.memory_stats(0)
    assert st["in_use"] == base and st["cached"] > 0
    mfs.release_cached_memory(0)
    assert mfs.memory_stats(0)["cached"] == 0
