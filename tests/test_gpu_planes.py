"""GPU parity of core marking on byte planes (more than eight axes, every span
below 2^15): edges of the 32-row tiles and 64-point runs, both plane depths,
the largest coordinates, pairs at exactly eps, passes that resume, and minPts
past the recorded neighbours, against the oracle's DBSCAN definition."""
from __future__ import annotations

import math

import numpy as np
import pytest

import oracle
from paper_1912_00323_amd.datagen import make_blobs, quantise

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    import torch
    assert torch.cuda.is_available(), "no HIP device visible"
    from paper_1912_00323_amd import hca
    c = hca.Context(0)
    yield c
    c.close()


def check(ctx, pts, eps, mp, tag):
    import torch
    print(f"[case] {tag} n={len(pts)} d={pts.shape[1]} eps={eps:.3f} minPts={mp}", flush=True)
    want, counts, _ = oracle.dbscan(pts, eps, mp, details=True)
    t = torch.from_numpy(np.ascontiguousarray(pts, np.int32)).cuda()
    got, core, st = ctx.cluster(t, eps, mp, core=True, stats=True)
    assert st["packed_rows"] == 1, tag
    assert np.array_equal(core.cpu().numpy().astype(bool), counts >= mp), tag
    assert np.array_equal(got.cpu().numpy(), want), tag


@pytest.mark.parametrize("d", [9, 31, 32, 33, 63, 64])
@pytest.mark.parametrize("budget", [None, "64", "192"])
def test_tile_edges(ctx, d, budget, monkeypatch):
    """One group of n points around the sizes of a tile, a run and a block of
    runs, every pair within reach of the other's list; then several groups."""
    if budget:
        monkeypatch.setenv("HCA_HD_BUDGET", budget)
    rng = np.random.default_rng(100 + d)
    for n in (31, 32, 33, 64, 65, 255, 257, 700):
        pts = rng.integers(-40, 41, size=(n, d)).astype(np.int32)
        typical = 40 * math.sqrt(2 * d / 3)
        for f, mp in ((0.8, 3), (1.0, 20)):
            check(ctx, pts, typical * f, mp, f"one group f={f} budget={budget}")
    pts = quantise(make_blobs(np.random.default_rng(d), 2500, d, 6, 0.03, 0.1), 10)
    for f, mp in ((0.75, 5), (0.95, 40)):
        check(ctx, pts, 0.03 * math.sqrt(2 * d) * f * 2 ** 10, mp, f"blobs f={f} budget={budget}")


def test_largest_coordinates(ctx):
    """One axis over the whole range of the byte split (span 2^15 - 1), far from
    zero, and pairs at exactly eps and one unit beyond."""
    rng = np.random.default_rng(5)
    base = np.array([-(1 << 20), 1 << 25], np.int64)
    for off in base:
        pts = rng.integers(0, 60, size=(900, 10)).astype(np.int64)
        pts[:, 3] = rng.choice([0, 1, 127, 128, 129, 16383, 16384, 32639, 32640, 32766, 32767], size=900)
        pts[0, 3], pts[1, 3] = 0, 32767
        pts = (pts + off).astype(np.int32)
        for eps in (60.0, 100.0, 16384.0, 40000.0):
            check(ctx, pts, eps, 6, f"whole range at {off}")
    # a lattice of spacing 5 along one axis and 12 along another: 5, 12 and
    # exactly 13 apart
    g = np.stack(np.meshgrid(np.arange(12) * 5, np.arange(12) * 12, indexing="ij"), -1).reshape(-1, 2)
    pts = np.zeros((len(g), 12), np.int32)
    pts[:, 2], pts[:, 9] = g[:, 0], g[:, 1]
    for eps in (4.99, 5.0, 12.0, 12.99, 13.0):
        check(ctx, pts, eps, 4, "lattice")
