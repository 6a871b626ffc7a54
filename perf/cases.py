"""Performance cases: the work a program does through this library's public
entry points, from a handful of probes to a 10M-query batch.

Every pass starts from points or a built tree and device queries and ends with
the caller's outputs: nearest neighbours (unbounded and within a radius),
range queries, a tree built and queried in one go, and many trees replayed as
one captured batch.  Sizes, distributions, list lengths and radii are those of
the repository's workloads (``datagen.py``, ``bench.py``) or generic ones
beside them; inputs are drawn on the device from the seed alone.
"""
from __future__ import annotations

import math

import torch

import paper_2210_12859_amd as kd

DEV = "cuda"
INF = math.inf


# ------------------------------------------------------------------ inputs

def _gen(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(int(seed))
    return g


def _mixture(n, dim, g, centers, sigma):
    lab = torch.randint(0, centers.shape[0], (n,), generator=g, device=DEV)
    x = torch.randn((n, dim), generator=g, device=DEV, dtype=torch.float32)
    return centers[lab] + sigma[lab, None] * x


def _centers(dist, dim, seed):
    """Cluster centres and widths of a distribution (the same for the points
    and the queries of one seed)."""
    g = _gen(seed * 7919 + 17)
    if dist == "gmm":  # 64 equal clusters, sigma 0.01
        c = torch.rand((64, dim), generator=g, device=DEV)
        return c, torch.full((64,), 0.01, device=DEV)
    c = torch.rand((256, dim), generator=g, device=DEV)
    lo, hi = math.log(0.002), math.log(0.05)
    return c, torch.exp(lo + (hi - lo) * torch.rand((256,), generator=g, device=DEV))


def _draw_points(dist, n, dim, seed, g):
    if dist == "uniform":
        return torch.rand((n, dim), generator=g, device=DEV)
    return _mixture(n, dim, g, *_centers(dist, dim, seed)).contiguous()


def _draw_queries(dist, n, dim, seed, g):
    x = _draw_points(dist, n, dim, seed, g)
    if dist == "clustered":  # one query in ten lies anywhere in the cube
        far = torch.rand((n,), generator=g, device=DEV) < 0.1
        x = torch.where(far[:, None], torch.rand((n, dim), generator=g, device=DEV), x)
    return x.contiguous()


def _inputs(case, seed):
    g = _gen(seed)
    pts = _draw_points(case["dist"], case["n"], case["dim"], seed, g)
    qs = _draw_queries(case["dist"], case["q"], case["dim"], seed, g)
    return pts, qs


def _batch_jobs(case):
    """(n, dim, dist, k) of each tree of a batch, from the case alone."""
    import random
    r = random.Random(case["jobs"] * 1000003 + case["n"])
    out = []
    for _ in range(case["jobs"]):
        n = int(round(math.exp(r.uniform(math.log(1000), math.log(case["n"])))))
        out.append((n, r.choice([2, 3, 4]), r.choice(["uniform", "gmm"]), r.choice([1, 8, 32])))
    return out


def _radius(dist, n, dim, mean):
    """Radius of a ball holding about `mean` points where the data is."""
    unit_ball = {2: math.pi, 3: 4.0 * math.pi / 3.0, 4: math.pi ** 2 / 2.0}[dim]
    vol = 1.0 if dist == "uniform" else 64.0 * (4.0 * math.pi) ** (dim / 2.0) * 0.01 ** dim
    return (mean * vol / (n * unit_ball)) ** (1.0 / dim)


# ------------------------------------------------------------------- cases

def _case(name, op, dist, dim, n, q, k=0, max_radius=0.0, mean=0.0, jobs=0):
    # max_radius 0: unbounded
    return dict(name=name, op=op, dist=dist, dim=dim, n=n, q=q, k=k, max_radius=max_radius, mean=mean, jobs=jobs)


def listed():
    return [
        # a few hundred interactive probes of a small scan: launches and latency
        _case("probe", "knn", "uniform", 3, 10_000, 250, k=8),
        # the headline size with the library's defaults: every point of a 1M cloud asks for 8 neighbours
        _case("knn8_1m", "knn", "uniform", 3, 1 << 20, 1 << 20, k=8),
        # the same call under the paper's own pruning rule (kd_opts.prune = 1), as the benchmark's headline runs it
        _case("paper_knn8_1m", "paper", "uniform", 3, 1 << 20, 1 << 20, k=8),
        # closest point of a registration step: one scan against a clustered model
        _case("fcp_gmm_1m", "fcp", "gmm", 3, 1 << 20, 1 << 20, k=1),
        # the large clustered workload, one query in ten far from the data
        _case("knn16_clustered_10m", "knn", "clustered", 3, 10_000_000, 10_000_000, k=16),
        # 4-D points and more queries than points (the shape of the paper's Table 1)
        _case("knn8_4d", "knn", "uniform", 4, 1 << 20, 4_000_000, k=8),
        # long lists inside a radius over ragged 2-D data: density estimates
        _case("knn50_2d_r", "knn", "gmm", 2, 200_003, 150_001, k=50, max_radius=0.01),
        # learned initial radius, a model trained beforehand
        _case("learned_knn8", "learned", "uniform", 3, 500_000, 700_001, k=8),
        # neighbours within a radius, the nearest 8 kept
        _case("ball8_1m", "ball", "uniform", 3, 1 << 20, 1 << 20, k=8, mean=8.0),
        # every point inside a box around each query, offsets and indices
        _case("boxes_all", "box_all", "gmm", 3, 400_000, 300_007, mean=48.0),
        # a new cloud: build its tree and ask for 8 neighbours of every point (normals of a frame)
        _case("frame_300k", "frame", "uniform", 3, 300_000, 300_000, k=8),
        # 96 trees of 1K to 200K points, 2-D to 4-D, k in {1, 8, 32}, replayed as one captured batch
        _case("batch_96", "batch", "mixed", 0, 200_000, 0, jobs=96),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case of the ranges above: sizes over their logarithm, every
    dimension, list lengths 1..64, bounded and unbounded radii."""
    op = rng.choice(["knn", "knn", "knn", "fcp", "paper", "learned", "ball", "box_all", "frame", "batch"])
    if op == "batch":
        return _case("", op, "mixed", 0, _log_int(rng, 5_000, 200_000), 0, jobs=rng.randint(3, 96))
    dim = 3 if op == "learned" else rng.choice([2, 3, 3, 4])
    dist = rng.choice(["uniform", "gmm"] if op in ("ball", "box_all", "learned") else ["uniform", "gmm", "clustered"])
    k = 1
    if op in ("knn", "paper", "learned", "frame"):
        k = rng.choice([1, 2, 4, 5, 8, 8, 10, 16, 20, 32, 50, 64])
    # the work of a query grows with its list and with the dimension; the
    # paper's rule visits far more nodes on clustered data
    top = 2_000_000 // (1 + k // 8) // (2 if dim == 4 else 1)
    if op == "paper" and dist != "uniform":
        top //= 16
    n = _log_int(rng, 1_000, 2_000_000 if op != "frame" else 1_000_000)
    q = n if op == "frame" else _log_int(rng, 200, top)
    if op == "frame":
        k = min(k, 10)
    if op == "ball":
        return _case("", op, dist, dim, n, q, k=rng.randint(1, 32), mean=float(rng.randint(2, 64)))
    if op == "box_all":
        return _case("", op, dist, dim, n, min(q, 1_000_000), mean=float(rng.randint(2, 64)))
    max_radius = 0.0
    if op in ("knn", "fcp", "paper") and rng.random() < 0.3:
        max_radius = round(rng.uniform(0.005, 0.05), 4)
    return _case("", op, dist, dim, n, q, k=k, max_radius=max_radius)


def _bound(case):
    return case["max_radius"] if case["max_radius"] > 0.0 else INF


def prepare(case, seed):
    """Device inputs and the tree (batch: the captured pipeline, learned: the
    trained model) a program keeps between calls."""
    if case["op"] == "batch":
        # every job's results in one pair of arrays, each job's rows from a
        # multiple of 64 elements on
        g = _gen(seed)
        meta = _batch_jobs(case)
        starts, total = [], 0
        for n, _, _, k in meta:
            starts.append(total)
            total += (n * k + 63) // 64 * 64
        idx = torch.full((total,), -1, dtype=torch.int32, device=DEV)
        d2 = torch.full((total,), INF, dtype=torch.float32, device=DEV)
        jobs = []
        for i, (n, dim, dist, k) in enumerate(meta):
            pts = _draw_points(dist, n, dim, seed * 131 + i, g)
            qs = _draw_queries(dist, n, dim, seed * 131 + i, g)
            a = starts[i]
            jobs.append(dict(tree=kd.kd_build(pts), queries=qs, k=k, out_idx=idx[a:a + n * k], out_d2=d2[a:a + n * k]))
        return dict(case=case, idx=idx, d2=d2, batch=kd.Batch(jobs))
    pts, qs = _inputs(case, seed)
    st = dict(case=case, queries=qs)
    if case["op"] == "frame":
        st["points"] = pts
        return st
    st["tree"] = kd.kd_build(pts)
    if case["op"] == "learned":
        train = _draw_queries(case["dist"], 65_536, case["dim"], seed, _gen(seed + 1_000_003))
        st["model"] = kd.kd_radius_model_train(st["tree"], train, case["k"], epochs=4)
    if case["op"] == "ball":
        st["radius"] = _radius(case["dist"], case["n"], case["dim"], case["mean"])
    if case["op"] == "box_all":
        half = 0.5 * (case["mean"] * (1.0 if case["dist"] == "uniform" else
                                      64.0 * (4.0 * math.pi) ** (case["dim"] / 2.0) * 0.01 ** case["dim"])
                      / case["n"]) ** (1.0 / case["dim"])
        st["lo"], st["hi"] = (qs - half).contiguous(), (qs + half).contiguous()
        # the program's neighbour buffer, of a fixed capacity
        st["kept"] = torch.full((int(case["q"] * case["mean"] * 1.5) + 65_536,), -1, dtype=torch.int32, device=DEV)
    return st


def run(state):
    """One pass; returns every output tensor of the call."""
    case = state["case"]
    op = case["op"]
    if op == "knn":
        return kd.kd_knn(state["tree"], state["queries"], case["k"], _bound(case))
    if op == "fcp":
        return kd.kd_fcp(state["tree"], state["queries"], _bound(case))
    if op == "paper":
        return kd.kd_knn_ex(state["tree"], state["queries"], case["k"], _bound(case), opts={"prune": 1})[:2]
    if op == "learned":
        return kd.kd_knn_learned(state["tree"], state["model"], state["queries"], case["k"], _bound(case))[:2]
    if op == "ball":
        return kd.kd_radius_search(state["tree"], state["queries"], state["radius"], cap=case["k"])
    if op == "box_all":
        kept = state["kept"]
        offsets, idx = kd.kd_box_search_all(state["tree"], state["lo"], state["hi"])
        m = min(idx.shape[0], kept.shape[0])
        kept[:m].copy_(idx[:m])
        return offsets, kept
    if op == "frame":
        tree = kd.kd_build(state["points"])
        out = kd.kd_knn(tree, state["queries"], case["k"], _bound(case))
        tree.close()
        return out
    state["batch"].run()
    return state["idx"], state["d2"]


def work(case):
    """Bytes: points and queries read once, results written once (a new tree's
    records once too).  Flops: the distance of every reported neighbour plus
    one comparison per tree level."""
    if case["op"] == "batch":
        b = f = 0
        for n, dim, _, k in _batch_jobs(case):
            b += n * dim * 4 * 2 + n * k * 8
            f += n * (k * (3 * dim - 1) + math.log2(n))
        return {"bytes": int(b), "flops": int(f)}
    n, q, dim = case["n"], case["q"], case["dim"]
    k = case["mean"] if case["op"] == "box_all" else case["k"]
    b = (n + q) * dim * 4
    if case["op"] == "box_all":
        b += q * dim * 4 + q * 8 + q * k * 4
    else:
        b += q * k * 8 + (q * 4 if case["op"] == "ball" else 0)
    if case["op"] == "frame":
        b += n * (dim + 1) * 4
    return {"bytes": int(b), "flops": int(q * (k * (3 * dim - 1) + math.log2(max(2, n))))}


def exact(case, seed):
    """Squared distances in 64 bits by direct comparison of every pair, for
    cases small enough; indices and counts are whole numbers."""
    op, n, q, dim = case["op"], case["n"], case["q"], case["dim"]
    if op in ("box_all", "batch") or n * q > 4_000_000_000:
        return None
    pts, qs = _inputs(case, seed)
    k = case["k"]
    r = _radius(case["dist"], n, dim, case["mean"]) if op == "ball" else _bound(case)
    # the bound as the call takes it: the square of the radius in 32 bits
    r32 = torch.tensor(r, dtype=torch.float32)
    bound = float(r32 * r32)
    p64 = pts.double()
    out = torch.full((q, k), INF, dtype=torch.float64, device=DEV)
    step = max(1, 64_000_000 // n)
    kk = min(k, n)
    for a in range(0, q, step):
        qq = qs[a:a + step].double()
        d2 = torch.zeros((qq.shape[0], n), dtype=torch.float64, device=DEV)
        for j in range(dim):
            dx = qq[:, j:j + 1] - p64[None, :, j]
            d2 += dx * dx
        out[a:a + step, :kk] = torch.topk(d2, kk, dim=1, largest=False, sorted=True).values
    out[out > bound * (1.0 + 1e-7)] = INF
    if op == "fcp" or (op != "ball" and k == 1):
        out = out[:, 0]
    return (None, None, out) if op == "ball" else (None, out)
