"""GPU parity of calls that follow others of the same shape on one context:
what a call returns or refuses does not depend on the calls before it."""
from __future__ import annotations

import numpy as np
import pytest

import oracle
from test_gpu import ctx, gpu_labels  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("small", ["0", None])
@pytest.mark.parametrize("d", [3, 8])
def test_other_radius_after_equal_boxes(ctx, d, small, monkeypatch):  # noqa: F811
    """Two calls on a wide box arm planning ahead from it; a call with a radius
    whose keys would not fit that box, but fit its own, is clustered, and one
    whose own keys do not fit is refused."""
    from paper_1912_00323_amd import hca
    if small:
        monkeypatch.setenv("HCA_SMALL", small)
    rng = np.random.default_rng(d)
    n, span, eps = 2000, (1 << 29 if d == 3 else 1 << 14), (1e6 if d == 3 else 4000.0)
    wide = rng.integers(0, span, size=(n, d)).astype(np.int32)
    line = np.zeros((n, d), np.int32)
    line[:, 0] = rng.permutation(n) * 10
    for _ in range(2):
        for _ in range(2):
            assert np.array_equal(gpu_labels(ctx, wide, eps, 3), oracle.dbscan(wide, eps, 3))
        assert np.array_equal(gpu_labels(ctx, line, 10.0, 3), oracle.dbscan(line, 10.0, 3))
    for _ in range(3):
        gpu_labels(ctx, wide, eps, 3)
    with pytest.raises(hca.HcaError) as e:
        gpu_labels(ctx, wide, 1.0, 3)
    assert e.value.status == hca.HCA_E_RANGE


@pytest.mark.parametrize("n,d", [(900, 2), (4000, 5), (2000, 8), (700, 16)])
def test_small_calls_with_changing_boxes(ctx, n, d):  # noqa: F811
    """Small calls whose box repeats and then differs: the labels stand, and up
    to eight axes the calls are counted as those of any size."""
    rng = np.random.default_rng(n)
    base = rng.integers(0, 1000, size=(n, d)).astype(np.int32)
    eps = 90.0 * d ** 0.5
    ctx.set_plan_reuse(True)
    gpu_labels(ctx, np.zeros((n + 1, d), np.int32), eps, 3)              # another shape: disarmed
    c0, r0 = ctx.plan_reuse_counts()
    want = []
    for shift in (0, 0, 0, 7, 7, 7, 0):
        pts = base.copy()
        pts[::3] += shift
        want.append((shift, oracle.dbscan(pts, eps, 3)))
        assert np.array_equal(gpu_labels(ctx, pts, eps, 3), want[-1][1]), shift
    c1, r1 = ctx.plan_reuse_counts()
    assert (c1 - c0, r1 - r0) == ((4, 2) if d <= 8 else (0, 0))
