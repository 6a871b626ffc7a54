"""Long radius and box calls (64 queries to a wave): counts, rows and the
variable-length results, order included, equal to the lane-by-lane kernel, which
a `visited` buffer or fewer than 20,000 queries select."""
import math

import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def _kd():
    import paper_2210_12859_amd as kd
    return kd


def _gen(seed):
    g = torch.Generator(device="cuda:0")
    g.manual_seed(seed)
    return g


def _mixture(g, n, dim):
    mean = torch.rand((40, dim), generator=g, device="cuda:0")
    pick = torch.randint(0, 40, (n,), generator=g, device="cuda:0")
    return mean[pick] + 0.01 * torch.randn((n, dim), generator=g, device="cuda:0")


def _same(a, b, what):
    for x, y in zip(a, b):
        assert (x is None) == (y is None), what
        if x is not None:
            assert torch.equal(x.view(torch.int32) if x.dtype == torch.float32 else x,
                               y.view(torch.int32) if y.dtype == torch.float32 else y), what


def _in_parts(call, q, part=10000):
    offs, idx, base = [torch.zeros(1, dtype=torch.int64, device="cuda:0")], [], 0
    for a in range(0, q, part):
        o, i = call(slice(a, min(q, a + part)))
        offs.append(o[1:] + base)
        base += int(o[-1])
        idx.append(i)
    return torch.cat(offs), torch.cat(idx)


def _check(tree, Q, r, what, caps=(0, 8), every=True):
    kd = _kd()
    print(f"[gpu] range packets {what}", flush=True)
    Q = Q.contiguous()
    vis = torch.empty(len(Q), dtype=torch.int32, device="cuda:0")
    lo, hi = (Q - r).contiguous(), (Q + r).contiguous()
    for cap in caps:
        _same(kd.kd_radius_search(tree, Q, r, cap=cap), kd.kd_radius_search(tree, Q, r, cap=cap, visited=vis),
              f"{what} ball cap={cap}")
        _same(kd.kd_box_search(tree, lo, hi, cap=cap), kd.kd_box_search(tree, lo, hi, cap=cap, visited=vis),
              f"{what} box cap={cap}")
    if every:
        _same(kd.kd_radius_search_all(tree, Q, r),
              _in_parts(lambda s: kd.kd_radius_search_all(tree, Q[s].contiguous(), r), len(Q)), f"{what} balls")
        _same(kd.kd_box_search_all(tree, lo, hi),
              _in_parts(lambda s: kd.kd_box_search_all(tree, lo[s].contiguous(), hi[s].contiguous()), len(Q)),
              f"{what} boxes")


# one leaf of up to six levels; root groups of 1 to 5 levels; three group levels
@pytest.mark.parametrize("dim", [2, 3, 4])
@pytest.mark.parametrize("n", [1, 2, 31, 32, 33, 63, 64, 65, 129, 1057, 2112, 4224, 8449, 9999])
def test_group_edges(dim, n):
    kd = _kd()
    g = _gen(n * 8 + dim)
    tree = kd.kd_build(torch.rand((n, dim), generator=g, device="cuda:0"))
    for q in (20000, 20001 + 64):
        Q = torch.rand((q, dim), generator=g, device="cuda:0") * 1.2 - 0.1
        _check(tree, Q, 0.5 * n ** (-1.0 / dim), f"D={dim} N={n} Q={q}")


@pytest.mark.parametrize("dim", [2, 3, 4])
@pytest.mark.parametrize("cap", [1, 2, 3, 5, 8, 9, 16, 20, 31, 32, 33, 64])
def test_list_lengths(dim, cap):
    kd = _kd()
    g = _gen(cap * 8 + dim)
    n = 15000
    for name, P, Q in (("uniform", torch.rand((n, dim), generator=g, device="cuda:0"),
                        torch.rand((2 * n + cap, dim), generator=g, device="cuda:0")),
                       ("mixture", _mixture(g, n, dim), _mixture(g, 2 * n + cap, dim))):
        _check(kd.kd_build(P), Q, 0.02 if name == "uniform" else 0.005, f"{name} D={dim} cap={cap}", (cap,), False)


@pytest.mark.parametrize("dim", [2, 3, 4])
def test_odd_regions(dim):
    """Ties on a grid, equal points, radius 0 and without a bound, NaN and
    infinite queries, empty and unbounded boxes, a far outlier, tiny and huge
    coordinates, both split rules."""
    kd = _kd()
    g = _gen(dim)
    q = 25000
    grid = torch.randint(0, 9, (9000, dim), generator=g, device="cuda:0").float()
    Q = torch.randint(0, 18, (q, dim), generator=g, device="cuda:0").float() / 2
    for split in (kd.KD_SPLIT_LEVEL, kd.KD_SPLIT_WIDEST):
        tree = kd.kd_build(grid, split=split)
        for r in (0.0, 0.5, 1.0):
            _check(tree, Q, r, f"ties D={dim} r={r} split={split}")
    _check(kd.kd_build(torch.full((500, dim), 0.25, device="cuda:0")), Q, 0.5, f"equal points D={dim}")
    P = torch.rand((9000, dim), generator=g, device="cuda:0")
    P[:3] = 1.0e6
    Q = torch.rand((q, dim), generator=g, device="cuda:0")
    bad = torch.randperm(q, generator=g, device="cuda:0")[:600]
    Q[bad[:100], 0] = math.nan
    Q[bad[100:200], dim - 1] = math.inf
    Q[bad[200:300]] = -math.inf
    Q[bad[300:400]] = 3.0e38
    Q[bad[400:500]] = 1.0e6
    tree = kd.kd_build(P)
    _check(tree, Q, 0.03, f"odd queries D={dim}")
    small = kd.kd_build(P[:50].contiguous())
    _check(small, Q, math.inf, f"no bound D={dim}", (0, 8, 20))
    for scale in (1.0e-37, 1.0e-25, 1.0e-18, 1.0e18, 1.0e30):
        _check(kd.kd_build((P[3:] * scale).contiguous()), torch.rand((q, dim), generator=g, device="cuda:0") * scale,
               0.03 * scale, f"scale {scale} D={dim}")
    # boxes: reversed, NaN, unbounded sides
    lo, hi = (Q - 0.02).contiguous(), (Q + 0.02).contiguous()
    lo[bad[500:520]] += 1.0
    lo[bad[520:540], 0] = math.nan
    hi[bad[540:560], 0] = math.inf
    lo[bad[560:580], dim - 1] = -math.inf
    vis = torch.empty(q, dtype=torch.int32, device="cuda:0")
    for cap in (0, 8):
        _same(kd.kd_box_search(tree, lo, hi, cap=cap), kd.kd_box_search(tree, lo, hi, cap=cap, visited=vis),
              f"odd boxes D={dim}")
    _same(kd.kd_box_search_all(tree, lo, hi),
          _in_parts(lambda s: kd.kd_box_search_all(tree, lo[s].contiguous(), hi[s].contiguous()), q),
          f"odd boxes, all, D={dim}")


@pytest.mark.parametrize("dim,n,q", [(2, 400000, 300000), (2, 400000, 299999), (3, 400000, 300000), (3, 300000, 300000),
                                     (3, 300001, 149999), (4, 500000, 500000), (4, 250000, 250000), (4, 250001, 250000)])
def test_line_of_the_route(dim, n, q):
    kd = _kd()
    g = _gen(q + n)
    tree = kd.kd_build(_mixture(g, n, dim))
    _check(tree, _mixture(g, q, dim), 0.002, f"line D={dim} N={n} Q={q}")
