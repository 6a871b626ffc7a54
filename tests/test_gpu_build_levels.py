"""GPU builder at the edges of its stages: trees of one workgroup (up to 2047
points), one to ten top levels, more than ten (lists grouped twice).  Bar: the
permutation equals the host builder's, and results and per-query visit counts
under both rules, which read every record and box reached, equal the host
tree's."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def _check(P, what, queries=4000):
    import paper_2210_12859_amd as kd
    print(f"[gpu] build {what}", flush=True)
    g = kd.kd_build(torch.from_numpy(P).to("cuda:0"))
    h = kd.kd_build_host(P)
    assert np.array_equal(g.order(), h.order()), what
    rng = np.random.default_rng(len(P))
    Q = P[rng.integers(0, len(P), queries)] + rng.normal(0, 1e-3, (queries, P.shape[1])).astype(np.float32)
    q = torch.from_numpy(np.ascontiguousarray(Q)).to("cuda:0")
    for prune in (1, 2):
        a = kd.kd_knn_ex(g, q, 4, want_visited=True, opts=dict(prune=prune))
        b = kd.kd_knn_ex(h, q, 4, want_visited=True, opts=dict(prune=prune))
        for x, y in zip(a, b):
            assert torch.equal(x.view(torch.int32), y.view(torch.int32)), (what, prune)
    assert g.info()["lo"] == h.info()["lo"] and g.info()["hi"] == h.info()["hi"], what
    g.close()
    h.close()


@pytest.mark.parametrize("dim", [2, 3, 4])
@pytest.mark.parametrize("n", [1, 2, 3, 63, 64, 65, 1023, 1024, 1535, 2046, 2047, 2048, 2049, 3071, 3072, 4095, 4096,
                               8191, 8192, 12345, 65535, 65536, 98304, 524287, 524288, 786433])
def test_sizes(dim, n):
    rng = np.random.default_rng(n * 4 + dim)
    _check(rng.random((n, dim), dtype=np.float32), f"D={dim} n={n}")


@pytest.mark.parametrize("dim,n", [(3, 1048576), (2, 2097151), (3, 2097151), (3, 2097152), (4, 2097152), (3, 2097153),
                                   (2, 3145728), (3, 4194304), (3, 5000001)])
def test_grouped_twice(dim, n):
    rng = np.random.default_rng(n + dim)
    _check(rng.random((n, dim), dtype=np.float32), f"D={dim} n={n}")


@pytest.mark.parametrize("dim", [2, 3, 4])
@pytest.mark.parametrize("n", [3000, 100000, 2200000])
def test_ties(dim, n):
    """Few distinct coordinates (ties by index), and one value per dimension."""
    rng = np.random.default_rng(n + dim)
    _check(rng.integers(-3, 4, (n, dim)).astype(np.float32), f"grid D={dim} n={n}", 64)
    if n < 1000000:
        _check(np.full((n, dim), -0.5, np.float32), f"equal D={dim} n={n}", 64)
