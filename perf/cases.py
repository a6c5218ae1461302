"""Clustering jobs that stand for the use of this library, for timing it.

Every job goes through the public binding: one call on device points (plain,
without allocation, or from host memory), a batch of data sets through one
call or a batch handle, and a burst of requests through the request server.
The data are Gaussian blobs over uniform noise in the unit cube, quantised to
fixed point, as in the generators of the package, drawn on the device from the
seed alone.
"""
import math
import random
from fractions import Fraction

import numpy as np
import torch

from paper_1912_00323_amd import hca

DEVICE = "cuda:0"


# ---------------------------------------------------------------------------
# the cases
# ---------------------------------------------------------------------------
def single(name, entry, n, d, blobs, std, eps, min_pts, q, noise, sizes="equal", core=False, merge="exact"):
    """One data set: n points in d axes, `blobs` blobs with standard deviations
    spread evenly over the logarithm from std[0] to std[1], a share `noise` of
    uniform points, radius eps (of the unit cube), 2^-q units."""
    case = {"entry": entry, "n": n, "d": d, "blobs": blobs, "std_lo": std[0], "std_hi": std[1], "eps": eps,
            "min_pts": min_pts, "q": q, "noise": noise, "sizes": sizes, "core": core, "merge": merge}
    return {"name": name, **case} if name else case


def several(name, entry, sets, n_lo, n_hi, dims, shape_seed):
    """Data sets of one shape: rows log-uniform in [n_lo, n_hi], axes from
    `dims`, and each set's own radius, minPts, blobs and noise, all fixed by
    shape_seed (the points are not)."""
    case = {"entry": entry, "sets": sets, "n_lo": n_lo, "n_hi": n_hi, "dims": dims, "shape_seed": shape_seed}
    return {"name": name, **case} if name else case


def high_eps(d):
    """Three quarters of the typical distance between two points of a blob of
    standard deviation 0.02 in d axes."""
    return 0.015 * math.sqrt(2.0 * d)


def listed():
    narrow = (0.02, 0.02)
    mixed = (0.005, 0.03)
    return [
        # the smallest of the paper's data sets (Leaf, 340 x 16): a call that
        # is all latency
        single("leaf_16d_340", "cluster", 340, 16, 20, narrow, high_eps(16), 10, 12, 0.05),
        # an interactive or per-frame call on a small planar point set
        single("blobs2d_10k", "cluster", 10_000, 2, 5, (0.03, 0.03), 0.02, 4, 12, 0.05),
        # a serving loop that must not allocate, a ragged size
        single("noalloc2d_100003", "noalloc", 100_003, 2, 30, mixed, 0.012, 6, 14, 0.10),
        # the benchmark's workload
        single("blobs2d_1m", "cluster", 1_000_000, 2, 50, (0.002, 0.01), 0.004, 8, 16, 0.10, "dirichlet"),
        # a large planar set (geographic positions), bound by memory
        single("blobs2d_16m", "cluster", 16_000_000, 2, 50, (0.002, 0.01), 0.004, 8, 16, 0.10, "dirichlet"),
        # a point cloud that lies in host memory
        single("host3d_177491", "host", 177_491, 3, 17, mixed, 0.017, 8, 14, 0.10),
        # one large request of the served workload's 5-axis kind
        single("served5d_1200017", "cluster", 1_200_017, 5, 16, mixed, 0.0175, 8, 14, 0.10),
        # the benchmark's second workload
        single("blobs8d_500k", "cluster", 500_000, 8, 20, narrow, 0.06, 10, 12, 0.05),
        # a motion-capture set (Vicon, 5045 x 27), with the core points asked for
        single("vicon_27d_5045", "cluster", 5_045, 27, 20, narrow, high_eps(27), 10, 12, 0.05, core=True),
        # the largest of the paper's data sets (PAMAP2, 3850505 x 54)
        single("pamap_54d_3850505", "cluster", 3_850_505, 54, 20, narrow, high_eps(54), 10, 12, 0.05),
        # the batched workload: many uneven data sets of one shape, through a
        # handle that plans once and replays a graph (the default knobs, so
        # that the times do not hang on what an autotuner chose)
        several("batch256", "batch", 256, 1_000, 200_000, "2,3,4", 4),
        # the served workload: requests of all sizes that arrive together
        several("server40", "server", 40, 10_000, 2_000_000, "2,3,5", 5),
    ]


def log_uniform(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng: random.Random):
    kind = rng.random()
    if kind < 0.12:
        return several("", rng.choice(["batch", "cluster_batch"]), rng.randint(3, 128), 1_000, 200_000, "2,3,4",
                       rng.randrange(1 << 30))
    if kind < 0.22:
        return several("", "server", rng.randint(3, 40), 10_000, 2_000_000, "2,3,5", rng.randrange(1 << 30))
    blobs, noise, min_pts = rng.randint(3, 30), rng.uniform(0.05, 0.15), rng.randint(4, 12)
    core = rng.random() < 0.25
    if kind < 0.42:
        # many axes
        d = rng.choice([9, 10, 12, 16, 21, 27, 33, 54, 64])
        n = log_uniform(rng, 300, 600_000)
        return single("", "cluster", n, d, blobs, (0.02, 0.02), high_eps(d), min_pts, 12, noise, core=core)
    if kind < 0.57:
        d = rng.choice([5, 5, 6, 7, 8])
        n = log_uniform(rng, 1_000, 1_200_000)
        if d == 5:
            return single("", "cluster", n, d, blobs, (0.005, 0.03), rng.uniform(0.01, 0.03), min_pts, 14, noise,
                          core=core)
        return single("", "cluster", n, d, blobs, (0.02, 0.02), high_eps(d), min_pts, 12, noise, core=core)
    entry = rng.choice(["cluster", "cluster", "cluster", "noalloc", "host"])
    d = rng.choice([1, 2, 2, 2, 3, 3, 4])
    most = 200_000 if entry == "noalloc" else 2_000_000 if entry == "host" else (16_000_000 if d <= 2 else 2_000_000)
    n = log_uniform(rng, 100, most)
    merge = "representatives" if entry == "cluster" and rng.random() < 0.1 else "exact"
    return single("", entry, n, d, blobs, (0.005, 0.03), rng.uniform(0.005, 0.03), min_pts, rng.choice([12, 14, 16]),
                  noise, rng.choice(["equal", "dirichlet"]), core=core and entry == "cluster", merge=merge)


def shapes(case):
    """The data sets of a case, as single cases."""
    if "sets" not in case:
        return [case]
    rng = random.Random(case["shape_seed"])
    dims = [int(v) for v in case["dims"].split(",")]
    return [single("", "cluster", log_uniform(rng, case["n_lo"], case["n_hi"]), rng.choice(dims), rng.randint(3, 30),
                   (0.005, 0.03), rng.uniform(0.005, 0.03), rng.randint(4, 12), 14, rng.uniform(0.05, 0.15))
            for _ in range(case["sets"])]


# ---------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------
def points(case, gen):
    """int32 [n, d] on the device, in random order."""
    n, d, k = case["n"], case["d"], case["blobs"]
    opt = {"dtype": torch.float64, "device": DEVICE, "generator": gen}
    n_noise = int(round(case["noise"] * n))
    n_blob = n - n_noise
    centres = torch.rand(k, d, **opt)
    stds = torch.as_tensor(np.geomspace(case["std_lo"], case["std_hi"], k), device=DEVICE)
    if case["sizes"] == "dirichlet":
        cut = torch.cumsum(-torch.log(torch.rand(k, **opt).clamp_min(1e-300)), 0)
        which = torch.searchsorted(cut / cut[-1], torch.rand(n_blob, **opt)).clamp_max(k - 1)
    else:
        which = torch.randint(0, k, (n_blob,), device=DEVICE, generator=gen)
    blob = centres[which] + stds[which, None] * torch.randn(n_blob, d, **opt)
    x = torch.cat([blob, torch.rand(n_noise, d, **opt)])[torch.randperm(n, device=DEVICE, generator=gen)]
    return torch.floor(x * float(2 ** case["q"]) + 0.5).to(torch.int32).contiguous()


def radius(case):
    return case["eps"] * 2 ** case["q"]


_kept = {}


def kept(what, make):
    """The contexts and the server that a program makes once and keeps."""
    if what not in _kept:
        _kept[what] = make()
    return _kept[what]


def approximate_context():
    ctx = hca.Context(0)
    ctx.set_exact(False)
    return ctx


def prepare(case, seed):
    gen = torch.Generator(device=DEVICE)
    gen.manual_seed(int(seed))
    sets = shapes(case)
    pts = [points(c, gen) for c in sets]
    state = {"case": case, "eps": [radius(c) for c in sets], "min_pts": [c["min_pts"] for c in sets], "points": pts}
    entry = case["entry"]
    if entry == "host":
        state["points"] = [pts[0].cpu().numpy()]
        return state
    rows, dims = [c["n"] for c in sets], [c["d"] for c in sets]
    state["rows"], state["dims"] = rows, dims
    if entry == "cluster":
        if case["merge"] != "exact":
            kept("approximate", approximate_context)
        return state
    # the caller's label arrays, one after the other
    state["labels"] = torch.empty(sum(rows), dtype=torch.int32, device=DEVICE)
    state["views"] = list(torch.split(state["labels"], rows))
    if entry == "batch":
        state["handle"] = hca.Batch(hca.context(0), rows, dims, state["eps"], state["min_pts"], tune=0)
    elif entry == "cluster_batch":
        state["points"] = [torch.cat([p.reshape(-1) for p in pts])]
    elif entry == "server":
        kept("server", lambda: hca.Server(0, workers=2, budget_bytes=48 << 30, max_batch=64, batch_ms=4.0))
    return state


def run(state):
    case, pts = state["case"], state["points"]
    entry = case["entry"]
    if entry == "cluster":
        eps, min_pts = state["eps"][0], state["min_pts"][0]
        if case["merge"] != "exact":
            return _kept["approximate"].cluster(pts[0], eps, min_pts, core=case["core"])
        return hca.cluster(pts[0], eps, min_pts, core=case["core"])
    if entry == "host":
        return hca.context(0).cluster_host(pts[0], state["eps"][0], state["min_pts"][0])
    if entry == "noalloc":
        return hca.context(0).cluster_noalloc(pts[0], state["eps"][0], state["min_pts"][0], state["labels"])
    if entry == "batch":
        state["handle"].run(pts, state["views"])
        return state["labels"]
    if entry == "cluster_batch":
        return hca.context(0).cluster_batch(pts[0], state["rows"], state["dims"], state["eps"], state["min_pts"],
                                            out=state["labels"])
    server = _kept["server"]
    for tag, (p, out) in enumerate(zip(pts, state["views"])):
        server.submit(p, state["eps"][tag], state["min_pts"][tag], out, tag)
    server.drain()
    failed = [tag for tag, status, _ in server.poll() if status != hca.HCA_OK]
    if failed:
        raise RuntimeError(f"requests {failed} failed")
    return state["labels"]


def work(case):
    """Each coordinate read and each label (and core flag) written once.  How
    many pair distances have to be taken depends on the method (points of a
    dense cube need none), so none are counted."""
    sets = shapes(case)
    return {"bytes": float(sum(c["n"] * (4 * c["d"] + 4 + (1 if c["core"] else 0)) for c in sets)), "flops": 0.0}


def exact(case, seed):
    """The same clustering from its definition, all pairs in 64-bit integers;
    None where there are too many pairs."""
    if "sets" in case or case["n"] > 12_000 or case["merge"] != "exact":
        return None
    gen = torch.Generator(device=DEVICE)
    gen.manual_seed(int(seed))
    x = points(case, gen).to(torch.int64)
    n, eps2 = case["n"], math.floor(Fraction(radius(case)) ** 2)
    near = torch.empty((n, n), dtype=torch.bool, device=DEVICE)
    best = torch.empty(n, dtype=torch.int64, device=DEVICE)
    far = torch.iinfo(torch.int64).max
    index = torch.arange(n, device=DEVICE)

    def dist2(i):
        t = torch.zeros((min(n, i + 1024) - i, n), dtype=torch.int64, device=DEVICE)
        for k in range(case["d"]):
            t += (x[i:i + 1024, k, None] - x[None, :, k]) ** 2
        return t

    for i in range(0, n, 1024):
        near[i:i + 1024] = dist2(i) <= eps2
    core = near.sum(1) >= case["min_pts"]
    # each core point takes the smallest component number in reach until
    # nothing changes
    comp = torch.where(core, index, n)
    while True:
        new = comp.clone()
        for i in range(0, n, 1024):
            reach = torch.where(near[i:i + 1024] & core, comp, n).min(1).values
            new[i:i + 1024] = torch.where(core[i:i + 1024], torch.minimum(comp[i:i + 1024], reach), n)
        new = torch.where(core, new[new.clamp_max(n - 1)], n)
        if torch.equal(new, comp):
            break
        comp = new
    # border points join their nearest core point, ties to the smaller index
    for i in range(0, n, 1024):
        best[i:i + 1024] = torch.where(near[i:i + 1024] & core, dist2(i) * n + index, far).min(1).values
    owner = torch.where(core, comp, torch.where(best < far, comp[best % n], n))
    first = torch.full((n + 1,), n, device=DEVICE).scatter_reduce(0, owner, index, "amin")
    order = torch.sort(first[:n][first[:n] < n]).values
    labels = torch.searchsorted(order, first[owner.clamp_max(n)]) if len(order) else torch.zeros_like(owner)
    labels = torch.where(owner < n, labels, -1).to(torch.int32)
    if case["entry"] == "host":
        return labels.cpu().numpy()
    return (labels, core.to(torch.uint8)) if case["core"] else labels
