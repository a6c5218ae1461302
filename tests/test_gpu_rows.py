"""GPU parity past eight axes of the walks over packed rows beside the tiles:
points alone in their groups, minPts 1 and 2, group counts on both sides of the
rule between the two, and groups around the chunks of the group boxes."""
from __future__ import annotations

import math

import numpy as np
import pytest

import oracle
from paper_1912_00323_amd.datagen import make_blobs, quantise
from test_gpu import ctx, gpu_labels  # noqa: F401

pytestmark = pytest.mark.gpu


def check(ctx, pts, eps, mp, tag):
    print(f"[case] {tag} n={len(pts)} d={pts.shape[1]} eps={eps:.2f} minPts={mp}", flush=True)
    want, counts, _ = oracle.dbscan(pts, eps, mp, details=True)
    got, core, st = gpu_labels(ctx, pts, eps, mp, core=True, stats=True)
    assert st["packed_rows"] == 1, tag
    assert np.array_equal(core.astype(bool), counts >= mp), tag
    assert np.array_equal(got, want), tag
    return st


@pytest.mark.parametrize("d", [9, 27, 54])
def test_rows_and_tiles(ctx, d):  # noqa: F811
    rng = np.random.default_rng(d)
    ratios = []
    for share in (0.0, 0.1, 0.3, 0.6, 1.0):
        # lone points, and a share of them in clumps of eight
        lone = rng.integers(0, 1 << 12, size=(2400, d))
        k = int(share * 2400) // 8 * 8
        lone[:k] = np.repeat(lone[:k:8], 8, 0) + rng.integers(-6, 7, size=(k, d))
        pts = np.clip(lone, 0, None)[rng.permutation(2400)].astype(np.int32)
        for mp in (1, 2, 8):
            st = check(ctx, pts, 9.0 * math.sqrt(d), mp, f"share {share}")
        ratios.append(2400 / st["n_groups"])
    assert min(ratios) < 1.25 < max(ratios), ratios
    for n in (15, 16, 17, 63, 64, 65, 1000):
        pts = quantise(make_blobs(np.random.default_rng(n), n, d, 2, 0.02, 0.1), 11)
        check(ctx, pts, 0.02 * math.sqrt(2 * d) * 0.8 * 2 ** 11, 4, "chunks")
