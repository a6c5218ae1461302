"""GPU parity of small calls, which are clustered by all pairs: against the
oracle's DBSCAN definition and against the general path (HCA_SMALL=0), at the
edges of words, waves and blocks, for every dimension and arithmetic, with the
data that the path has to leave to the general one, and with plan reuse.  A
few tests of the general path run here without the all-pairs path."""
from __future__ import annotations

import math

import numpy as np
import pytest

import oracle
import test_gpu
import test_gpu_highd
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


def run(ctx, pts, eps, mp):
    import torch
    lab, core = ctx.cluster(torch.from_numpy(np.ascontiguousarray(pts, np.int32)).cuda(), eps, mp, core=True)
    return lab.cpu().numpy(), core.cpu().numpy().astype(bool)


def check(ctx, pts, eps, mp, tag):
    print(f"[case] {tag} n={len(pts)} d={pts.shape[1]} eps={eps:.3f} minPts={mp}", flush=True)
    want, counts, _ = oracle.dbscan(pts, eps, mp, details=True)
    lab, core = run(ctx, pts, eps, mp)
    assert np.array_equal(core, counts >= mp), tag
    assert np.array_equal(lab, want), tag


@pytest.mark.parametrize("d", [1, 2, 3, 4, 5, 8, 9, 32, 33, 64])
def test_edges(ctx, d):
    """Point counts around a word, a wave, a slice and a block of points; few
    neighbours and many, minPts 1 and past n."""
    for n in (1, 2, 31, 33, 63, 64, 65, 255, 257, 1023, 1025, 2100):
        pts = quantise(make_blobs(np.random.default_rng(7 * n + d), n, d, 4, 0.03, 0.15), 10)
        typical = 0.03 * math.sqrt(2 * d) * 2 ** 10
        for f, mp in ((0.35, 3), (0.8, 6), (6.0, 12), (0.5, 1), (1.0, n + 1)):
            check(ctx, pts, typical * f, mp, f"edges f={f}")


@pytest.mark.parametrize("d", [1, 2, 3, 8])
def test_wide_distances(ctx, d, monkeypatch):
    """Squared distances past 31 bits, spans up to 2^30 - 1; what the general
    path refuses (cube keys past 63 bits) is refused."""
    from paper_1912_00323_amd import hca
    rng = np.random.default_rng(d)
    pts = rng.integers(-(1 << 28), 1 << 28, size=(700, d)).astype(np.int32)
    pts[:350] = pts[350:] + rng.integers(-3000, 3001, size=(350, d))
    pts[0], pts[1] = -(1 << 29), (1 << 29) - 1
    for eps, mp in ((2500.0, 2), (1e7, 3), (4e8, 5)):
        try:
            with monkeypatch.context() as m:
                m.setenv("HCA_SMALL", "0")
                run(ctx, pts, eps, mp)
        except hca.HcaError as refused:
            with pytest.raises(hca.HcaError) as e:
                run(ctx, pts, eps, mp)
            assert e.value.status == refused.status == hca.HCA_E_RANGE
            continue
        check(ctx, pts, eps, mp, "wide")


def test_ties_chains_and_duplicates(ctx):
    """Border points between clusters (ties to the smaller index), a chain whose
    forest is deep, and points that are all the same."""
    rng = np.random.default_rng(4)
    line = np.stack([np.arange(3000) * 10, np.zeros(3000)], 1).astype(np.int32)
    for order in (np.arange(3000), np.arange(3000)[::-1], rng.permutation(3000)):
        check(ctx, line[order], 10.0, 3, "chain")
    grid = np.stack(np.meshgrid(np.arange(40), np.arange(40)), -1).reshape(-1, 2).astype(np.int32) * 7
    pts = np.concatenate([np.repeat(grid[::9], 4, 0), grid])[rng.permutation(len(grid) + 4 * len(grid[::9]))]
    for eps, mp in ((7.0, 7), (9.9, 9), (14.0, 14)):
        check(ctx, pts, eps, mp, "ties")
    check(ctx, np.full((4000, 3), 5, np.int32), 1.0, 4000, "duplicates")


def test_same_as_the_general_path(ctx, monkeypatch):
    """Sizes up to the path's limits and past them, against the general path;
    data past eight axes that byte planes do not hold, and keys past 63 bits,
    come out (or are refused) as before, however often they are called."""
    from paper_1912_00323_amd import hca
    rng = np.random.default_rng(1)
    for n, d, eps, q in ((9000, 1, 3.0, 14), (12288, 2, 300.0, 14), (12289, 2, 300.0, 14), (16384, 3, 300.0, 14),
                         (16000, 4, 250.0, 14), (12000, 6, 250.0, 12), (16384, 12, 300.0, 12), (9001, 40, 400.0, 12),
                         (3000, 12, 6000.0, 17), (5000, 20, 900.0, 14)):
        pts = quantise(make_blobs(rng, n, d, 9, 0.02, 0.1, "dirichlet"), q)
        got = [run(ctx, pts, eps, 8) for _ in range(2)]
        with monkeypatch.context() as m:
            m.setenv("HCA_SMALL", "0")
            want = run(ctx, pts, eps, 8)
        for lab, core in got:
            assert np.array_equal(lab, want[0]) and np.array_equal(core, want[1]), (n, d)
    far = np.zeros((50, 8), np.int32)
    far[0] = (1 << 30) - 1
    for _ in range(3):
        with pytest.raises(hca.HcaError) as e:
            run(ctx, far, 3.0, 2)
        assert e.value.status == hca.HCA_E_RANGE
    far[0] = np.iinfo(np.int32).max
    far[1] = np.iinfo(np.int32).min
    with pytest.raises(hca.HcaError) as e:
        run(ctx, far, 1e9, 2)
    assert e.value.status == hca.HCA_E_RANGE


# the general path at small sizes
@pytest.fixture
def general(monkeypatch):
    monkeypatch.setenv("HCA_SMALL", "0")


def test_general_small_workload(ctx, general):
    test_gpu.test_small_workload(ctx)


@pytest.mark.parametrize("d", [1, 2, 3, 4, 5, 6, 7, 8, 12, 54])
def test_general_path(ctx, general, d):
    for n in (1, 65, 3000):
        pts = quantise(make_blobs(np.random.default_rng(50 + d + n), n, d, 5, 0.03, 0.1), 10)
        for f, mp in ((0.5, 3), (0.9, 8)):
            check(ctx, pts, 0.03 * math.sqrt(2 * d) * f * 2 ** 10, mp, f"general f={f}")


def test_general_plan_reuse(ctx, general):
    test_gpu.test_plan_reuse(ctx)


def test_general_degenerate_many_axes(ctx, general):
    test_gpu_highd.test_degenerate_many_axes(ctx)
