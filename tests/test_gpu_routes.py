"""Calls on both sides of the lines between the kNN kernels, against the oracle:
one wave per query up to the line, packets of 64 sorted queries (or the lanes)
above it.  The stage timers tell which kernels ran: only calls with one wave per
query as they come have no sort."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

# the longest call of one wave per query, by dimension and list size
LINE = {(2, 8): 65536, (2, 16): 98304, (2, 32): 131072, (3, 8): 98304, (3, 16): 131072, (3, 32): 262144,
        (4, 8): 131072, (4, 16): 163840, (4, 32): 262144, (2, 64): 327680, (3, 64): 327680, (4, 64): 327680}


def _data(rng, n, dim):
    """Half uniform, half in narrow clusters: queries with few and with many
    candidates share packets."""
    mean = rng.random((32, dim), dtype=np.float32)
    x = mean[rng.integers(0, 32, n)] + 0.003 * rng.standard_normal((n, dim)).astype(np.float32)
    some = rng.random(n) < 0.5
    x[some] = rng.random((int(some.sum()), dim), dtype=np.float32)
    return np.ascontiguousarray(x, np.float32)


def _call(kd, tree, Qs, k, r=np.inf):
    """Rows and the number of sort stages of one call."""
    q = torch.from_numpy(Qs).to("cuda:0")
    kd.kd_timing_enable(True)
    try:
        for stage in ("sort", "traverse"):
            kd.kd_timing_collect(stage)
        i, d = kd.kd_knn(tree, q, k, r)
        torch.cuda.synchronize()
        sorts = kd.kd_timing_collect("sort")[1]
        kd.kd_timing_collect("traverse")
    finally:
        kd.kd_timing_enable(False)
    return i.cpu().numpy(), d.cpu().numpy(), sorts


@pytest.mark.parametrize("dim", [3, 4])
@pytest.mark.parametrize("k", [1, 2, 4, 7, 8, 16, 27])
def test_packet_rows(oracle_lib, dim, k):
    """Every list size of the packets, lanes without a candidate among them (the
    bytes these read name no entry outside the chunks held)."""
    import paper_2210_12859_amd as kd
    rng = np.random.default_rng(dim * 64 + k)
    q = LINE[(dim, 8 if k <= 8 else (16 if k <= 16 else 32))] + 77
    P, Qs = _data(rng, 60000, dim), _data(rng, q, dim)
    print(f"[gpu] packet rows D={dim} k={k} Q={q}", flush=True)
    tree = kd.kd_build(torch.from_numpy(P).to("cuda:0"))
    order = oracle_lib.build_tree(P)
    for r in (np.inf, 0.02):
        i, d, sorts = _call(kd, tree, Qs, k, r)
        assert sorts == 1
        ri, rd, _ = oracle_lib.knn(P, order, Qs, k, r)
        assert np.array_equal(i.reshape(ri.shape), ri)
        assert np.array_equal(d.reshape(rd.shape).view(np.uint32), rd.view(np.uint32))


@pytest.mark.parametrize("dim,k", sorted(LINE))
def test_lines(oracle_lib, dim, k):
    """The longest call without a sort, and one more query."""
    import paper_2210_12859_amd as kd
    rng = np.random.default_rng(dim * 64 + k)
    q = LINE[(dim, k)]
    P, Qs = _data(rng, 50000, dim), _data(rng, q + 1, dim)
    print(f"[gpu] line D={dim} k={k} Q={q}", flush=True)
    tree = kd.kd_build(torch.from_numpy(P).to("cuda:0"))
    ri, rd, _ = oracle_lib.knn(P, oracle_lib.build_tree(P), Qs, k)
    for n, sorted_ in ((q, 0), (q + 1, 1)):
        i, d, sorts = _call(kd, tree, Qs[:n], k)
        assert sorts == sorted_
        assert np.array_equal(i, ri[:n]) and np.array_equal(d.view(np.uint32), rd[:n].view(np.uint32))


def test_tuned_trees_keep_the_kernels(oracle_lib):
    """Options tuned where calls go lane by lane (or set by the caller) leave
    small calls to one wave per query; rows are the oracle's throughout."""
    import paper_2210_12859_amd as kd
    rng = np.random.default_rng(7)
    P, Qs = _data(rng, 1_000_000, 3), _data(rng, 110_000, 3)  # above the line, too sparse for packets
    order = oracle_lib.build_tree(P)
    ri, rd, _ = oracle_lib.knn(P, order, Qs, 8)
    set_tree, tuned_tree = (kd.kd_build(torch.from_numpy(P).to("cuda:0")) for _ in range(2))
    lanes = dict(block=512, lds_levels=0, sort_bits=24, waves_per_cu=16, heavy_trips=0, prune=2)
    kd.kd_tree_set_tuned(set_tree, 8, lanes)
    best, _ = kd.kd_autotune(tuned_tree, torch.from_numpy(Qs).to("cuda:0"), 8)
    assert kd.kd_tree_get_tuned(set_tree, 8) == lanes and kd.kd_tree_get_tuned(tuned_tree, 8) == best
    for tree in (set_tree, tuned_tree):
        for q, sorted_ in ((250, 0), (20_000, 0), (110_000, 1)):
            print(f"[gpu] tuned Q={q}", flush=True)
            i, d, sorts = _call(kd, tree, Qs[:q], 8)
            assert sorts == sorted_
            assert np.array_equal(i, ri[:q]) and np.array_equal(d.view(np.uint32), rd[:q].view(np.uint32))


def test_batch_options_make_the_kept_plan_again():
    """A group that kept one wave per query: a batch made from the options that
    the tuner returned takes them too (lane by lane a replay takes 10 times as
    long), and tuning leaves no batch slower."""
    import paper_2210_12859_amd as kd
    g = torch.Generator(device="cuda:0")
    g.manual_seed(3)
    jobs = []
    for i in range(8):
        tree = kd.kd_build(torch.rand((10000, 3), generator=g, device="cuda:0"))
        q = torch.rand((250, 3), generator=g, device="cuda:0")
        jobs.append(dict(tree=tree, queries=q, k=8, out_idx=torch.empty((250, 8), dtype=torch.int32, device="cuda:0"),
                         out_d2=torch.empty((250, 8), dtype=torch.float32, device="cuda:0")))

    def ms(b):
        best = np.inf
        for _ in range(10):
            e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            e0.record()
            b.run()
            e1.record()
            torch.cuda.synchronize()
            best = min(best, e0.elapsed_time(e1))
        return best

    print("[gpu] batch options", flush=True)
    b = kd.Batch(jobs)
    t_default = ms(b)
    rows = [j["out_idx"].clone() for j in jobs]
    chosen = b.autotune(reps=1)
    assert len(chosen) == 1
    again, lanes = kd.Batch(jobs, opts=chosen[0]), kd.Batch(jobs, opts=dict(block=512))
    t_tuned, t_again, t_lanes = ms(b), ms(again), ms(lanes)
    print(f"[gpu] default {t_default:.4f} tuned {t_tuned:.4f} again {t_again:.4f} lanes {t_lanes:.4f} ms", flush=True)
    assert t_tuned < 0.5 * t_lanes and t_again < 0.5 * t_lanes
    again.run()
    torch.cuda.synchronize()
    assert all(torch.equal(j["out_idx"], r) for j, r in zip(jobs, rows))


@pytest.mark.parametrize("q,stats", [(300, False), (300, True), (120_000, False), (400_000, False), (400_000, True)])
def test_models_cost_nothing_where_rows_do_not_need_them(oracle_lib, q, stats):
    """Calls with a model take the kernels of kd_knn; the model runs where
    statistics ask for it, or the call goes lane by lane (120,000 queries over 1M
    points)."""
    import paper_2210_12859_amd as kd
    rng = np.random.default_rng(q)
    n = 1_000_000 if q == 120_000 else 300_000
    P, Qs = _data(rng, n, 3), _data(rng, q, 3)
    g = torch.from_numpy(Qs).to("cuda:0")
    tree = kd.kd_build(torch.from_numpy(P).to("cuda:0"))
    model = kd.kd_radius_model_train(tree, torch.from_numpy(_data(rng, 4096, 3)).to("cuda:0"), 8, epochs=1)
    print(f"[gpu] model route q={q} stats={stats}", flush=True)
    kd.kd_timing_enable(True)
    try:
        kd.kd_timing_collect("mlp")
        i, d = kd.kd_knn_learned(tree, model, g, 8, want_stats=stats)[:2]
        torch.cuda.synchronize()
        runs = kd.kd_timing_collect("mlp")[1]
        for stage in ("sort", "traverse"):
            kd.kd_timing_collect(stage)
    finally:
        kd.kd_timing_enable(False)
    assert (runs > 0) == (stats or q == 120_000)
    ri, rd, _ = oracle_lib.knn(P, oracle_lib.build_tree(P), Qs, 8)
    assert np.array_equal(i.cpu().numpy().reshape(ri.shape), ri)
    assert np.array_equal(d.cpu().numpy().reshape(rd.shape).view(np.uint32), rd.view(np.uint32))


def _uniform(dim, n, q, seed):
    g = torch.Generator(device="cuda:0")
    g.manual_seed(seed)
    return torch.rand((n, dim), generator=g, device="cuda:0"), torch.rand((q, dim), generator=g, device="cuda:0")


@pytest.mark.parametrize("dim,k,n,line", [(3, 1, 200_000, 450_000), (3, 8, 300_000, 287_500), (4, 16, 262_144, 282_768),
                                          (3, 32, 400_000, 350_000)])
@pytest.mark.parametrize("host", [False, True])
def test_even_points_line(dim, k, n, line, host):
    """Both sides of the packets' line over evenly spread points (trees packed on
    either side) equal the lane-by-lane kernel."""
    import paper_2210_12859_amd as kd
    P, Q = _uniform(dim, n, line, k)
    tree = kd.kd_build_host(P.cpu().numpy()) if host else kd.kd_build(P)
    for q in (line - 1, line):
        print(f"[gpu] even line D={dim} k={k} Q={q} host={host}", flush=True)
        i, d = kd.kd_knn(tree, Q[:q], k)
        ri, rd, _ = kd.kd_knn_ex(tree, Q[:q], k, opts={"prune": 2})
        assert torch.equal(i, ri) and torch.equal(d.view(torch.int32), rd.view(torch.int32))


@pytest.mark.parametrize("host", [False, True])
def test_even_points_are_not_slower_than_lane_by_lane(host):
    """200,000 queries over 1M uniform points, k = 16: packets take 1.5 times as
    long as the lanes."""
    import paper_2210_12859_amd as kd
    P, Q = _uniform(3, 1_000_000, 200_000, 1)
    tree = kd.kd_build_host(P.cpu().numpy()) if host else kd.kd_build(P)

    def ms(**kw):
        best = np.inf
        for _ in range(20):
            e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            e0.record()
            kd.kd_knn_ex(tree, Q, 16, **kw)
            e1.record()
            torch.cuda.synchronize()
            best = min(best, e0.elapsed_time(e1))
        return best

    default, lanes = ms(), ms(opts={"prune": 2})
    print(f"[gpu] even points host={host}: default {default:.3f} lanes {lanes:.3f} ms", flush=True)
    assert default < 1.25 * lanes


@pytest.mark.parametrize("below", [0, 1])
def test_batch_line_of_closest_points(below):
    """A 3-D class of closest points on the packets' density, and one query below."""
    import paper_2210_12859_amd as kd
    jobs, want = [], []
    for i, n in enumerate((40_000, 120_000, 80_001)):
        q = n - n // 4 - (below if i == 1 else 0)
        P, Q = _uniform(3, n, q, i)
        tree = kd.kd_build(P)
        want.append(kd.kd_knn_ex(tree, Q, 1, opts={"prune": 2})[:2])
        jobs.append(dict(tree=tree, queries=Q, k=1, out_idx=torch.full((q,), -7, dtype=torch.int32, device="cuda:0"),
                         out_d2=torch.full((q,), -7.0, dtype=torch.float32, device="cuda:0")))
    print(f"[gpu] batch line below={below}", flush=True)
    b = kd.Batch(jobs)
    for _ in range(3):
        b.run()
        torch.cuda.synchronize()
        for j, (wi, wd) in zip(jobs, want):
            assert torch.equal(j["out_idx"], wi.view(-1)) and torch.equal(j["out_d2"], wd.view(-1))
            j["out_idx"].fill_(-7)
    b.close()
