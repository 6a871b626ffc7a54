"""Variable-length range results: what they keep alive, and calls whose first
guess finds no memory."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("q,half", [(1, 0.01), (5000, 0.0), (5000, 0.02), (5000, 0.05), (70000, 0.0), (70000, 0.01), (70000, 0.05)])
def test_results_keep_what_they_hold(oracle_lib, q, half, monkeypatch):
    """At most twice the result, or 4 MiB, with and without memory for the
    guess."""
    import paper_2210_12859_amd as kd
    rng = np.random.default_rng(q)
    P, C = rng.random((100000, 3), dtype=np.float32), rng.random((q, 3), dtype=np.float32)
    lo, hi = C - np.float32(half), C + np.float32(half)
    tree = kd.kd_build(torch.from_numpy(P).to("cuda:0"))
    count = oracle_lib.box(P, lo, hi)[0].astype(np.int64)
    want = np.concatenate([[0], np.cumsum(count)])
    tlo, thi = torch.from_numpy(lo).to("cuda:0"), torch.from_numpy(hi).to("cuda:0")
    print(f"[gpu] range memory q={q} half={half}", flush=True)
    offsets, idx = kd.kd_box_search_all(tree, tlo, thi)
    assert np.array_equal(offsets.cpu().numpy(), want) and idx.shape[0] == want[-1]
    assert idx.untyped_storage().nbytes() <= max(1 << 22, 2 * 4 * int(want[-1]))

    real = torch.empty

    def short(*args, **kw):
        if args[0] == 64 * q:
            raise torch.OutOfMemoryError("no memory for the guess")
        return real(*args, **kw)

    monkeypatch.setattr(torch, "empty", short)
    o2, i2 = kd.kd_box_search_all(tree, tlo, thi)
    assert torch.equal(o2, offsets) and torch.equal(i2, idx)
