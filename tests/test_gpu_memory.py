"""GPU parity where the device has no room for the larger workspaces
(HCA_ALLOC_LIMIT makes those allocations fail): calls that a smaller workspace
can serve are served, the others report HCA_E_NOMEM."""
from __future__ import annotations

import math

import numpy as np
import pytest

import oracle
from paper_1912_00323_amd.datagen import make_blobs, quantise

pytestmark = pytest.mark.gpu


def blobs(n, d, seed=1, q=12):
    return quantise(make_blobs(np.random.default_rng(seed), n, d, 5, 0.03, 0.1), q)


def smallest_limit(call):
    """The smallest of a series of limits (a quarter more each) at which the call
    is served, and its result there."""
    from paper_1912_00323_amd import hca
    limit = 1 << 16
    while True:
        try:
            return limit, call(limit)
        except hca.HcaError as e:
            assert e.status == hca.HCA_E_NOMEM, e
        limit += limit // 4


@pytest.mark.parametrize("n,d", [(8000, 1), (10_000, 2), (10_000, 20), (3000, 54)])
def test_single_calls(n, d, monkeypatch):
    """By all pairs or over the grid, with byte planes or without: no call needs
    more than the general path alone does (HCA_SMALL=0, HCA_PACKED=0)."""
    import torch
    from paper_1912_00323_amd import hca
    pts = blobs(n, d)
    eps = 0.03 * math.sqrt(2 * d) * 0.7 * 2 ** 12 if d > 1 else 20.0
    want = oracle.dbscan(pts, eps, 5)
    x = torch.from_numpy(np.ascontiguousarray(pts, np.int32)).cuda()

    def call(limit):
        monkeypatch.setenv("HCA_ALLOC_LIMIT", str(limit))
        ctx = hca.Context(0)
        try:
            return ctx.cluster(x, eps, 5).cpu().numpy()
        finally:
            ctx.close()
    with_all, got = smallest_limit(call)
    assert np.array_equal(got, want)
    monkeypatch.setenv("HCA_SMALL", "0")
    monkeypatch.setenv("HCA_PACKED", "0")
    general, got = smallest_limit(call)
    assert np.array_equal(got, want)
    print(f"[case] n={n} d={d}: served from {with_all} bytes on, general path {general}", flush=True)
    assert with_all <= general


def test_batches(monkeypatch):
    """3-D batches go back to prefix ranges of one axis."""
    import torch
    from paper_1912_00323_amd import hca
    sets = [blobs(n, 3, seed=n, q=14) for n in (60_000, 5000, 31_000)]
    eps, mps = [200.0, 300.0, 250.0], [5, 4, 6]
    want = [oracle.hca_grid(p, e, m, threads=8) for p, e, m in zip(sets, eps, mps)]
    pts = [torch.from_numpy(np.ascontiguousarray(p, np.int32)).cuda() for p in sets]
    rows, dims = [len(p) for p in sets], [3] * 3
    outs = [torch.empty(n, dtype=torch.int32, device="cuda") for n in rows]

    def handle(limit):
        monkeypatch.setenv("HCA_ALLOC_LIMIT", str(limit))
        ctx = hca.Context(0)
        b = None
        try:
            b = hca.Batch(ctx, rows, dims, eps, mps, tune=0)
            for _ in range(2):
                b.run(pts, outs)
            return [o.cpu().numpy() for o in outs]
        finally:
            if b is not None:
                b.close()
            ctx.close()

    def flat(limit):
        monkeypatch.setenv("HCA_ALLOC_LIMIT", str(limit))
        ctx = hca.Context(0)
        try:
            got = ctx.cluster_batch(torch.cat([p.reshape(-1) for p in pts]), rows, dims, eps, mps).cpu().numpy()
            return np.split(got, np.cumsum(rows)[:-1])
        finally:
            ctx.close()
    for call in (handle, flat):
        limit, got = smallest_limit(call)
        for g, w in zip(got, want):
            assert np.array_equal(g, w)
        monkeypatch.setenv("HCA_PREFIX", "0")
        without, _ = smallest_limit(call)
        monkeypatch.delenv("HCA_PREFIX")
        print(f"[case] batch served from {limit} bytes on, without ranges {without}", flush=True)
        assert limit <= 1.3 * without
