"""Batches at default options: classes answered in packets, one wave per query
(small batches) or lane by lane, every row bit-equal to the single-tree
lane-by-lane call (explicit options), on replays too."""
import math

import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def _gen(seed):
    g = torch.Generator(device="cuda:0")
    g.manual_seed(seed)
    return g


def _points(g, kind, n, dim):
    if kind == "uniform":
        return torch.rand((n, dim), generator=g, device="cuda:0")
    mean = torch.rand((32, dim), generator=g, device="cuda:0")
    pick = torch.randint(0, 32, (n,), generator=g, device="cuda:0")
    return mean[pick] + 0.01 * torch.randn((n, dim), generator=g, device="cuda:0")


def _run(specs, what, tune=False):
    import paper_2210_12859_amd as kd
    jobs, want = [], []
    for i, (kind, dim, n, q, k, r) in enumerate(specs):
        g = _gen(1000 * i + n + q)
        tree = kd.kd_build(_points(g, kind, n, dim))
        Q = _points(g, kind, q, dim)
        if q > 40:
            Q[::37, 0] = math.nan
            Q[5::41] = math.inf
            Q[7::43] += 20.0
        want.append(kd.kd_knn_ex(tree, Q, k, r, opts={"prune": 2})[:2])
        jobs.append(dict(tree=tree, queries=Q, k=k, max_radius=r,
                         out_idx=torch.full((q, k), -7, dtype=torch.int32, device="cuda:0"),
                         out_d2=torch.full((q, k), -7.0, dtype=torch.float32, device="cuda:0")))
    print(f"[gpu] batch {what} {len(jobs)} jobs", flush=True)
    b = kd.Batch(jobs)
    if tune:
        b.autotune(reps=1)
    for rep in range(3):
        for j in jobs:
            j["out_idx"].fill_(-7)
            j["out_d2"].fill_(-7.0)
        b.run()
        torch.cuda.synchronize()
        for i, (j, w) in enumerate(zip(jobs, want)):
            assert torch.equal(j["out_idx"].view(w[0].shape), w[0]), (what, rep, specs[i])
            assert torch.equal(j["out_d2"].view(w[1].shape).view(torch.int32), w[1].view(torch.int32)), (what, rep, specs[i])
    b.close()


INF = math.inf
SIZES = [(1, 1), (33, 64), (64, 65), (1057, 63), (1057, 1), (5000, 3001), (9000, 12000), (20000, 20000)]


@pytest.mark.parametrize("k", [1, 3, 8, 16, 20, 32, 64])
def test_small_batches(k):
    """Few queries in all: one wave each."""
    _run([(("uniform", "mixture")[i % 2], 2 + i % 3, n, min(q, 900), k, INF if i % 2 else 0.05)
          for i, (n, q) in enumerate(SIZES + SIZES[::-1] + SIZES[2:])], f"small k={k}")


@pytest.mark.parametrize("tune", [False, True])
def test_packets(tune):
    """More queries: 3-D and 4-D classes by packets (partial ones at the jobs'
    ends, k below the class's list), 2-D and long lists lane by lane."""
    specs = []
    for dim in (2, 3, 4):
        for k in (1, 2, 5, 8, 13, 32, 40):
            for i, (n, q) in enumerate(SIZES):
                specs.append((("uniform", "mixture")[(i + k) % 2], dim, n, q, k, INF if i % 3 else 0.02))
            specs.append(("mixture", dim, 20000, 29999, k, INF))
    _run(specs if not tune else specs[::3], f"packets tune={tune}", tune)


def test_class_with_a_sparse_job():
    """One job's queries too sparse for packets: its class stays with the lanes."""
    _run([("uniform", 3, 100000, 200000, 8, INF), ("mixture", 3, 200000, 3000, 8, INF),
          ("mixture", 4, 100000, 150000, 8, INF), ("uniform", 4, 50000, 70000, 7, 0.1)], "sparse job")
