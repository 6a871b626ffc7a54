"""One wave per query: rows bit-equal to the oracle's definition at the edges of
the groups (leaves of 5 and 6 levels, root groups of 1 to 5 levels), of the
list (1..64 lanes) and of the call sizes that take it."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def _kd():
    import paper_2210_12859_amd as kd
    return kd


def _t(a):
    return torch.from_numpy(np.ascontiguousarray(a)).to("cuda:0")


def _check(oracle_lib, P, Qs, k, r, what, split=0):
    kd = _kd()
    print(f"[gpu] wave {what}", flush=True)
    tree = kd.kd_build(_t(P), split=split)
    i, d = kd.kd_knn(tree, _t(Qs), k, r)
    ri, rd = oracle_lib.brute(P, Qs, k, r)
    assert np.array_equal(i.cpu().numpy().reshape(ri.shape), ri)
    assert np.array_equal(d.cpu().numpy().reshape(rd.shape).view(np.int32), rd.view(np.int32))


# one leaf; leaves of 5 / 6 levels; root groups of 1..5 levels above them
SIZES = [1, 2, 31, 32, 33, 63, 64, 65, 1055, 1056, 1057, 2112, 4224, 8447, 8449, 16897, 33793, 40000]


@pytest.mark.parametrize("dim", [2, 3, 4])
@pytest.mark.parametrize("n", SIZES)
def test_group_edges(oracle_lib, dim, n):
    rng = np.random.default_rng(dim * 100003 + n)
    P = rng.random((n, dim), dtype=np.float32)
    Qs = np.concatenate([rng.random((40, dim), dtype=np.float32), P[:8],
                         (10.0 * rng.standard_normal((6, dim))).astype(np.float32)])
    for k in (1, 8, 33, 64):
        _check(oracle_lib, P, Qs, k, np.inf, f"D={dim} N={n} k={k}")


@pytest.mark.parametrize("dim", [2, 3, 4])
@pytest.mark.parametrize("k", [1, 2, 16, 31, 32, 63, 64])
def test_ties_bounds_and_odd_queries(oracle_lib, dim, k):
    """Exact ties on an integer grid, duplicates, zero and finite radii, NaN
    and infinite queries, both split rules."""
    kd = _kd()
    rng = np.random.default_rng(dim * 31 + k)
    grid = rng.integers(0, 5, size=(3000, dim)).astype(np.float32)
    Qs = np.concatenate([grid[:30], grid[30:50] + np.float32(0.5), grid[50:60] - np.float32(7.0)])
    bad = Qs[:6].copy()
    bad[:3, 0] = np.nan
    bad[3:, -1] = np.inf
    Qs = np.concatenate([Qs, bad])
    for r in (np.inf, 1.0, 0.0):
        for split in (kd.KD_SPLIT_LEVEL, kd.KD_SPLIT_WIDEST):
            _check(oracle_lib, grid, Qs, k, r, f"ties D={dim} k={k} r={r} split={split}", split)


@pytest.mark.parametrize("dim,q", [(2, 65536), (2, 65537), (3, 131072), (3, 131073), (4, 131072), (4, 131073)])
def test_line_of_the_route(dim, q):
    """Both sides of the line equal the lane-by-lane kernel (explicit options)."""
    kd = _kd()
    g = torch.Generator(device="cuda:0")
    g.manual_seed(q)
    P = torch.rand((20000, dim), generator=g, device="cuda:0")
    Qs = torch.rand((q, dim), generator=g, device="cuda:0")
    tree = kd.kd_build(P)
    print(f"[gpu] wave line D={dim} Q={q}", flush=True)
    i, d = kd.kd_knn(tree, Qs, 5)
    ri, rd, _ = kd.kd_knn_ex(tree, Qs, 5, opts={"prune": 2})
    assert torch.equal(i, ri) and torch.equal(d.view(torch.int32), rd.view(torch.int32))
