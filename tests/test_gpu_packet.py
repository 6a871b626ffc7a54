"""Long calls (packets of 64 queries; lists over 32: one wave per query on the
sorted queries): every row bit-equal to the lane-by-lane kernel, which explicit
options select and which the parity tests hold to the oracle."""
import math

import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

LINE = {3: 131072, 4: 196608}  # calls of at most this many queries go one wave each


def _kd():
    import paper_2210_12859_amd as kd
    return kd


def _gen(seed):
    g = torch.Generator(device="cuda:0")
    g.manual_seed(seed)
    return g


def _mixture(g, n, dim, comps=48, width=0.01):
    mean = torch.rand((comps, dim), generator=g, device="cuda:0")
    pick = torch.randint(0, comps, (n,), generator=g, device="cuda:0")
    wide = width * torch.rand((comps, 1), generator=g, device="cuda:0")
    return mean[pick] + wide[pick] * torch.randn((n, dim), generator=g, device="cuda:0")


def _check(P, Q, k, what, r=math.inf, tree=None):
    kd = _kd()
    print(f"[gpu] packets {what}", flush=True)
    tree = kd.kd_build(P.contiguous()) if tree is None else tree
    Q = Q.contiguous()
    i, d = kd.kd_knn(tree, Q, k, r)
    ri, rd, _ = kd.kd_knn_ex(tree, Q, k, r, opts={"prune": 2})
    assert torch.equal(i, ri), what
    assert torch.equal(d.view(torch.int32), rd.view(torch.int32)), what


# leaves of 5 / 6 levels, no group above them, root groups of 1 to 5 levels
@pytest.mark.parametrize("dim", [3, 4])
@pytest.mark.parametrize("n", [1, 2, 31, 32, 33, 63, 64, 65, 1057, 4224, 8449, 33793])
def test_group_edges(dim, n):
    g = _gen(n * 8 + dim)
    P = torch.rand((n, dim), generator=g, device="cuda:0")
    for q in (LINE[dim] + 1, LINE[dim] + 64):
        Q = torch.rand((q, dim), generator=g, device="cuda:0") * 1.2 - 0.1
        for k in (1, 8):
            _check(P, Q, k, f"D={dim} N={n} Q={q} k={k}")


@pytest.mark.parametrize("dim", [3, 4])
@pytest.mark.parametrize("k", [1, 2, 3, 4, 5, 8, 13, 16, 17, 31, 32])
def test_list_lengths(dim, k):
    """Uniform and clustered data, finite and zero radii."""
    g = _gen(k * 8 + dim)
    q = 330000 + k
    for name, P, Q in (
        ("uniform", torch.rand((200003, dim), generator=g, device="cuda:0"),
         torch.rand((q, dim), generator=g, device="cuda:0")),
        ("mixture", _mixture(g, 200003, dim), _mixture(g, q, dim)),
    ):
        for r in (math.inf, 0.01, 0.0):
            _check(P, Q, k, f"{name} D={dim} k={k} r={r}", r)


@pytest.mark.parametrize("dim", [3, 4])
def test_odd_queries_and_points(dim):
    """Ties on an integer grid, all points equal, a far outlier that shares a
    packet's cell, queries far outside, NaN and infinite ones, and coordinates
    at both ends of the floats' range."""
    g = _gen(dim)
    q = LINE[dim] + 4321
    grid = torch.randint(0, 9, (20000, dim), generator=g, device="cuda:0").float()
    Q = torch.randint(0, 18, (q, dim), generator=g, device="cuda:0").float() / 2
    for k in (1, 8, 20):
        for r in (math.inf, 1.0, 0.0):
            _check(grid, Q, k, f"ties D={dim} k={k} r={r}", r)
    _check(torch.full((5000, dim), 0.25, device="cuda:0"), Q, 8, f"equal points D={dim}")
    P = torch.rand((50000, dim), generator=g, device="cuda:0")
    P[:4] = 1.0e6
    Q = torch.rand((q, dim), generator=g, device="cuda:0")
    bad = torch.randperm(q, generator=g, device="cuda:0")[:512]
    Q[bad[:64], 0] = math.nan
    Q[bad[64:128], dim - 1] = math.inf
    Q[bad[128:192]] = -math.inf
    Q[bad[192:256]] = 3.0e38
    Q[bad[256:320]] *= 1.0e7
    Q[bad[320:384]] = 1.0e6
    Q[bad[384:448]] += 50.0
    for k in (1, 8, 16):
        _check(P, Q, k, f"odd queries D={dim} k={k}")
        _check(P, Q, k, f"odd queries D={dim} k={k} r=0.05", 0.05)
    far = P.clone()
    far[:8] = 2.0e18  # outside the range the packets take
    _check(far, Q, 8, f"far points D={dim}")
    for scale in (1.0e-30, 1.0e-18, 1.0e-8, 1.0e8, 5.0e16, 1.0e17):
        Ps, Qs = P[4:] * scale, torch.rand((q, dim), generator=g, device="cuda:0") * scale
        _check(Ps, Qs, 8, f"scale {scale} D={dim}")
        _check(Ps + scale * 1000, Qs + scale * 1000, 4, f"shifted scale {scale} D={dim}")


def test_points_dropped_from_the_bound_walk():
    """4-D clusters of different widths: packets that straddle clusters drop
    points far from their middle, which must not shorten the bound."""
    g = _gen(3)
    P = _mixture(g, 200000, 4, comps=256, width=0.02)
    Q = _mixture(g, 1000000, 4, comps=256, width=0.02)
    same = torch.cat([P + 1.0e-4 * torch.randn(P.shape, generator=g, device="cuda:0"), Q[:300000]])
    for k in (8, 16):
        _check(P, Q, k, f"clusters k={k}")
        _check(P, same, k, f"clusters, near queries k={k}")


@pytest.mark.parametrize("dim,k,n,q", [(3, 8, 1048576, 131071), (3, 8, 1048584, 131073), (3, 1, 600000, 149999),
                                       (3, 1, 600000, 150000), (3, 32, 1200000, 299999), (3, 32, 1200000, 300000),
                                       (4, 8, 1000000, 249999), (4, 8, 1000000, 250000), (2, 8, 1000, 70000)])
def test_line_of_the_route(dim, k, n, q):
    """Both sides of where packets take over from the other kernels."""
    g = _gen(q)
    P = torch.rand((n, dim), generator=g, device="cuda:0")
    _check(P, torch.rand((q, dim), generator=g, device="cuda:0"), k, f"line D={dim} k={k} N={n} Q={q}")


@pytest.mark.parametrize("dim", [2, 3, 4])
@pytest.mark.parametrize("k", [33, 64])
def test_long_lists_sorted(dim, k):
    """Lists over 32: the caller's order up to 327,680 queries, sorted above."""
    kd = _kd()
    g = _gen(dim * 64 + k)
    P = torch.rand((30011, dim), generator=g, device="cuda:0")
    for split in (kd.KD_SPLIT_LEVEL, kd.KD_SPLIT_WIDEST):
        tree = kd.kd_build(P, split=split)
        for q in (327680, 327681):
            Q = torch.rand((q, dim), generator=g, device="cuda:0")
            Q[::1001, 0] = math.nan
            for r in (math.inf, 0.05):
                _check(P, Q, k, f"long lists D={dim} k={k} Q={q} r={r}", r, tree)


def test_widest_rule_and_streams():
    """The widest-rule tree keeps the lanes; two streams at once give what one
    gives."""
    kd = _kd()
    g = _gen(77)
    P = torch.rand((100000, 3), generator=g, device="cuda:0")
    Q = torch.rand((200000, 3), generator=g, device="cuda:0")
    _check(P, Q, 8, "widest", tree=kd.kd_build(P, split=kd.KD_SPLIT_WIDEST))
    tree = kd.kd_build(P)
    want = kd.kd_knn(tree, Q, 8)
    torch.cuda.synchronize()
    side = [torch.cuda.Stream(), torch.cuda.Stream()]
    got = []
    for rep in range(4):
        with torch.cuda.stream(side[rep % 2]):
            got.append(kd.kd_knn(tree, Q, 8))
    torch.cuda.synchronize()
    for i, d in got:
        assert torch.equal(i, want[0]) and torch.equal(d, want[1])


@pytest.mark.parametrize("k,margin", [(1, 0.1), (8, 0.1), (8, 0.0), (8, -0.5), (8, 3.0), (5, 0.1), (20, 0.1)])
def test_model_radii(k, margin):
    """Model radii start the packets: good ones, ones too small (lists left short,
    alone or many to a packet) and ones that reach too far."""
    kd = _kd()
    g = _gen(k)
    P = torch.cat([torch.rand((150000, 3), generator=g, device="cuda:0"), _mixture(g, 150000, 3)])
    Q = torch.cat([torch.rand((100001, 3), generator=g, device="cuda:0"), _mixture(g, 100000, 3)])
    Q[::5003, 1] = math.nan
    Q[1::5003] = math.inf
    Q[2::5003] += 30.0
    tree = kd.kd_build(P)
    m = kd.kd_radius_model_train(tree, Q[3:20003:1][torch.isfinite(Q[3:20003]).all(dim=1)].contiguous(), k, epochs=2)
    m = kd.kd_model_create(*m.params(), margin, k)
    for r in (math.inf, 0.02):
        print(f"[gpu] packets model k={k} margin={margin} r={r}", flush=True)
        i, d = kd.kd_knn_learned(tree, m, Q, k, r)[:2]
        ri, rd, _ = kd.kd_knn_ex(tree, Q, k, r, opts={"prune": 2})
        assert torch.equal(i.view(ri.shape), ri) and torch.equal(d.view(rd.shape).view(torch.int32), rd.view(torch.int32))
