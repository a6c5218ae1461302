"""Data of few cubes with very many points each, and other sets that are
cheap for the method: labels against the construction, and phases that must
not grow with the square of the points (their times stay far below what the
quadratic walk takes)."""
from __future__ import annotations

import numpy as np
import pytest

from test_gpu import ctx  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d,cubes", [(4, 8), (5, 2), (6, 2), (8, 1)])
def test_groups_of_one_huge_cube(ctx, d, cubes):  # noqa: F811
    """A million points in a few groups of a single cube: nothing to link inside
    a group (47 ms when its points were walked all the same)."""
    import torch
    n = 1_000_000
    gen = torch.Generator(device="cuda").manual_seed(d)
    which = torch.randint(0, cubes, (n,), device="cuda", generator=gen)
    pts = torch.randint(0, 3, (n, d), device="cuda", generator=gen)
    pts[:, 0] += 4000 * which
    pts = pts.to(torch.int32).contiguous()
    first = torch.full((cubes,), n, device="cuda").scatter_reduce(0, which, torch.arange(n, device="cuda"), "amin")
    want = torch.argsort(torch.argsort(first))[which].to(torch.int32)
    ctx.set_profiling("all")
    try:
        for _ in range(2):
            assert torch.equal(ctx.cluster(pts, 60.0, 8), want)
        times = ctx.phase_times()
    finally:
        ctx.set_profiling(None)
    print(times, flush=True)
    assert times["intra"] < 5.0, times


@pytest.mark.parametrize("d", [5, 6])
def test_long_lists_in_a_small_array(ctx, d, monkeypatch):  # noqa: F811
    """Lists longer than a wave's even share of the list array, with room for
    all of them together: they fit, and the labels are the oracle's."""
    import oracle
    from test_gpu import gpu_labels
    monkeypatch.setenv("HCA_LIST_SLAB", "64")
    rng = np.random.default_rng(d)
    eps = 100.0
    block = rng.integers(0, 300, size=(3000, d))
    block[:, 5:] //= 30
    lone = np.zeros((4000, d), np.int64)
    lone[:, 0], lone[:, 1] = 3000 + 400 * (np.arange(4000) % 64), 400 * (np.arange(4000) // 64)
    pts = np.concatenate([block, lone])[rng.permutation(7000)].astype(np.int32)
    want = oracle.dbscan(pts, eps, 5)
    got, st = gpu_labels(ctx, pts, eps, 5, stats=True)
    assert np.array_equal(got, want)
    assert st["list_overflow"] == 0, st


@pytest.mark.parametrize("slab", ["0", "16", None])
@pytest.mark.parametrize("budget", ["16", "256"])
def test_points_left_by_the_lanes(ctx, slab, budget, monkeypatch):  # noqa: F811
    """Core marking by eight lanes per point at small sizes: few and nearly all
    points left to the chunks, no lists, and lists that overflow."""
    import oracle
    from paper_1912_00323_amd.datagen import make_blobs, quantise
    from test_gpu import gpu_labels
    monkeypatch.setenv("HCA_SMALL", "0")
    monkeypatch.setenv("HCA_CORE_LANES", "1")
    monkeypatch.setenv("HCA_CORE_BUDGET", budget)
    if slab:
        monkeypatch.setenv("HCA_LIST_SLAB", slab)
    if budget == "16":
        monkeypatch.setenv("HCA_WAVE_BLOCKS", "8")          # many units per wave
    for d, std, f, mp in ((5, 0.03, 0.5, 4), (6, 0.2, 0.55, 9), (6, 0.01, 0.6, 40), (8, 0.02, 0.75, 10), (7, 0.3, 0.3, 2)):
        pts = quantise(make_blobs(np.random.default_rng(mp + d), 5003, d, 4, std, 0.15), 12)
        eps = std * np.sqrt(2 * d) * f * 2 ** 12
        print(f"[case] d={d} std={std} mp={mp} slab={slab} budget={budget}", flush=True)
        want, counts, _ = oracle.dbscan(pts, eps, mp, details=True)
        got, core = gpu_labels(ctx, pts, eps, mp, core=True)
        assert np.array_equal(core.astype(bool), counts >= mp), (d, mp)
        assert np.array_equal(got, want), (d, mp)


@pytest.mark.parametrize("n,eps,mp", [(1_600_000, 0.012, 4), (1_600_000, 0.03, 9), (1_600_000, 0.0012, 8)])
def test_planes_by_records_and_representatives(ctx, n, eps, mp):  # noqa: F811
    """Large planar sets on both sides of the rule between merging from records
    and by representatives, against the grid oracle."""
    import oracle
    import torch
    from paper_1912_00323_amd.datagen import make_blobs, quantise
    pts = quantise(make_blobs(np.random.default_rng(n + mp), n, 2, 30, 0.02, 0.1), 15)
    print(f"[case] eps={eps} mp={mp}", flush=True)
    got = ctx.cluster(torch.from_numpy(np.ascontiguousarray(pts, np.int32)).cuda(), eps * 2 ** 15, mp).cpu().numpy()
    assert np.array_equal(got, oracle.hca_grid(pts, eps * 2 ** 15, mp, threads=8))


@pytest.mark.parametrize("n", [6 << 20, 6_400_001])
def test_labels_in_and_out_of_order(ctx, n):  # noqa: F811
    """Binned labels where some tiles' points lie in order and write their
    labels at once, and others' do not, with core flags: the grid oracle's."""
    import oracle
    import torch
    rng = np.random.default_rng(n)
    pts = rng.integers(0, 1 << 15, size=(n, 2))
    pts[: n // 2] = (pts[: n // 2] // 800) * 800 + rng.integers(0, 60, size=(n // 2, 2))
    pts = pts[rng.permutation(n)]
    k = n // 3                                              # a third in the order of its cubes
    key = (pts[:k, 0] // 20) * 4096 + pts[:k, 1] // 20
    pts[:k] = pts[:k][np.argsort(key, kind="stable")]
    pts = np.ascontiguousarray(pts, np.int32)
    got, core = ctx.cluster(torch.from_numpy(pts).cuda(), 30.0, 12, core=True)
    want, flags, _ = oracle.hca_grid(pts, 30.0, 12, threads=8, details=True)
    assert np.array_equal(core.cpu().numpy(), flags.astype(np.uint8))
    assert np.array_equal(got.cpu().numpy(), want)
