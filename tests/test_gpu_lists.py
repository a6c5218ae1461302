"""GPU parity of the neighbour lists built from prefix ranges, several groups
per wave, against the oracle: group counts around the packs of a wave, ranges
that are narrowed along the next axis, and ranges too long to be scanned."""
from __future__ import annotations

import math

import numpy as np
import pytest

import test_gpu
from paper_1912_00323_amd.datagen import make_blobs, quantise
from test_gpu import ctx  # noqa: F401

pytestmark = pytest.mark.gpu


def lattice(rng, d, axes, per_axis, step):
    """Points scattered by up to step / 4 around a lattice over the last axes."""
    grid = np.stack(np.meshgrid(*[np.arange(per_axis)] * axes, indexing="ij"), -1).reshape(-1, axes) * step
    pts = rng.integers(0, step // 4 + 1, size=(2 * len(grid), d))
    pts[:, d - axes:] += np.repeat(grid, 2, 0)
    return pts[rng.permutation(len(pts))].astype(np.int32)


@pytest.mark.parametrize("d", [3, 4, 5, 6, 7, 8])
def test_prefix_packs(ctx, d, monkeypatch):  # noqa: F811
    monkeypatch.setenv("HCA_SMALL", "0")
    eps = 100.0
    for mode in ("cube", "group") if d < 5 else ("group",):
        monkeypatch.setenv("HCA_SEARCH", mode)
        # few groups: packs of a wave left part empty
        for n in (1, 3, 7, 8, 9, 64, 65, 700):
            rng = np.random.default_rng(31 * n + d)
            test_gpu.check(ctx, rng.integers(0, 700, size=(n, d)).astype(np.int32), eps, 2, f"{mode} few")
        # columns of more groups than a range is scanned whole, and planes of
        # more than are scanned at all
        for axes, per_axis in ((1, 900), (2, 45)):
            for step in (1.4 * eps, 0.75 * eps):
                rng = np.random.default_rng(axes + d)
                test_gpu.check(ctx, lattice(rng, d, axes, per_axis, int(step)), eps, 3, f"{mode} lattice {axes}")
        pts = quantise(make_blobs(np.random.default_rng(d), 4000, d, 5, 0.03, 0.2), 12)
        test_gpu.check(ctx, pts, 0.025 * math.sqrt(2 * d) * 2 ** 12, 5, f"{mode} blobs")


@pytest.mark.parametrize("budget", ["16", "256"])
def test_group_lanes(ctx, budget, monkeypatch):  # noqa: F811
    """Core marking by eight lanes per point: minPts below and above the lanes
    and the records of a point, budgets that leave most points to a wave, and
    groups of more than a chunk of points."""
    monkeypatch.setenv("HCA_SMALL", "0")
    monkeypatch.setenv("HCA_CORE_BUDGET", budget)
    for d in (6, 8):
        for std, mp in ((0.03, 3), (0.03, 14), (0.008, 40)):
            pts = quantise(make_blobs(np.random.default_rng(mp + d), 5003, d, 4, std, 0.15), 12)
            test_gpu.check(ctx, pts, 0.018 * math.sqrt(2 * d) * 2 ** 12, mp, f"lanes {budget}")


@pytest.mark.parametrize("d", [3, 4])
def test_cubes_joined_by_few_pairs(ctx, d, monkeypatch):  # noqa: F811
    """Cubes of core points only, no recorded neighbours, whose nearest point
    pairs lie just within or just past eps: the sampled pairs miss them, and
    small and large products of points take the lane and the worklist."""
    monkeypatch.setenv("HCA_SMALL", "0")
    monkeypatch.setenv("HCA_SEARCH", "cube")
    eps, rng = 100.0, np.random.default_rng(d)
    for lanes in ("1", "0"):
        monkeypatch.setenv("HCA_CORE_LANES", lanes)
        for size in (3, 4, 5, 40, 300):
            sets = []
            for pair in range(40):
                base = np.zeros(d, np.int64)
                base[d - 1] = 400 * pair
                for side in (0, 1):
                    clump = rng.integers(0, 30, size=(size, d))
                    clump[:, 0] += side * int(rng.integers(70, 131))
                    sets.append(clump + base)
            pts = np.concatenate(sets)
            pts = pts[rng.permutation(len(pts))].astype(np.int32)
            test_gpu.check(ctx, pts, eps, 3, f"few pairs {size}")


@pytest.mark.parametrize("d,n,eps,q", [(4, 1 << 18, 0.010, 14), (4, 1 << 18, 0.010, 16), (4, 300_001, 0.008, 12),
                                       (3, 20_001, 0.022, 14), (3, 99_999, 0.03, 16), (3, 100_000, 0.03, 12),
                                       (3, 200_000, 0.03, 14)])
def test_search_rules_agree(ctx, d, n, eps, q, monkeypatch):  # noqa: F811
    """Sizes and densities at which a call changes its search: the same labels
    and core points as cube by cube over lists."""
    import torch
    pts = quantise(make_blobs(np.random.default_rng(n), n, d, 9, 0.02, 0.15), q)
    x = torch.from_numpy(np.ascontiguousarray(pts, np.int32)).cuda()
    got = [t.cpu().numpy() for t in ctx.cluster(x, eps * 2 ** q, 6, core=True)]
    monkeypatch.setenv("HCA_SEARCH", "cube")
    want = [t.cpu().numpy() for t in ctx.cluster(x, eps * 2 ** q, 6, core=True)]
    assert np.array_equal(got[0], want[0]) and np.array_equal(got[1], want[1])


@pytest.mark.parametrize("d,n", [(1, 1_600_000), (2, 1_572_864), (2, 1_700_003)])
def test_large_planes_without_representatives(ctx, d, n, monkeypatch):  # noqa: F811
    """Large sets of one and two axes merge from recorded neighbours and
    sampled pairs: the same labels as with representatives (no records)."""
    import torch
    pts = quantise(make_blobs(np.random.default_rng(n), n, d, 40, 0.01, 0.1), 16)
    x = torch.from_numpy(np.ascontiguousarray(pts, np.int32)).cuda()
    for eps, mp in ((0.002, 8), (0.0005, 40)):
        got = ctx.cluster(x, eps * 2 ** 16, mp)
        monkeypatch.setenv("HCA_RECORD", "0")
        want = ctx.cluster(x, eps * 2 ** 16, mp)
        monkeypatch.delenv("HCA_RECORD")
        assert torch.equal(got, want), (d, n, eps)


@pytest.mark.parametrize("n", [(3 << 20) - 1, 3 << 20, (3 << 20) + 1, 3_300_000])
def test_labels_of_large_sets(ctx, n):  # noqa: F811
    """Labels and core flags binned by input position: they follow the points
    into another order, clusters numbered by their first points."""
    import torch
    gen = torch.Generator(device="cuda").manual_seed(n)
    x = torch.rand(n, 2, device="cuda", generator=gen)
    x[: n // 2] = (x[: n // 2] * 40).floor() / 40 + 0.004 * torch.randn(n // 2, 2, device="cuda", generator=gen)
    x = (x * 2 ** 15).to(torch.int32).contiguous()
    order = torch.randperm(n, device="cuda", generator=gen)
    eps, mp = 20.0, 12
    lab, core = ctx.cluster(x, eps, mp, core=True)
    lab2, core2 = ctx.cluster(x[order].contiguous(), eps, mp, core=True)
    assert torch.equal(core[order], core2)
    # one label per label where core points are concerned (a border point may
    # have cores of two clusters in reach, and goes to the first)
    c = core2.bool()
    a, b = lab[order][c].long(), lab2[c].long()
    assert int(a.min()) == 0 and int(b.min()) == 0 and int(a.max()) == int(b.max())
    pairs = torch.unique(torch.stack([a, b], 1), dim=0)
    assert len(pairs) == int(a.max()) + 1 == len(torch.unique(pairs[:, 1]))
    assert torch.equal(lab[order] < 0, lab2 < 0)
    # numbered by first member
    members = lab >= 0
    first = torch.full((int(lab.max()) + 1,), n, device="cuda").scatter_reduce(
        0, lab[members].long(), torch.arange(n, device="cuda")[members], "amin")
    assert bool((first[1:] > first[:-1]).all())
