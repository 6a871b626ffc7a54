"""Builds where memory is short: a cloud whose tree and order fit is built, with
the least workspace and the tree after it, to the same tree."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

N = 1 << 24
# bytes a point of the order and the larger of the tree and the least workspace
PEAK = {(2, 0): 36, (3, 0): 56, (4, 0): 68, (3, 1): 58}


@pytest.mark.parametrize("dim,split", sorted(PEAK))
def test_short_memory(dim, split):
    import paper_2210_12859_amd as kd
    g = torch.Generator(device="cuda:0")
    g.manual_seed(dim)
    P = torch.rand((N, dim), generator=g, device="cuda:0")
    Q = torch.rand((2000, dim), generator=g, device="cuda:0")
    tree = kd.kd_build(P, split=split)
    order, (wi, wd) = tree.order(), kd.kd_knn(tree, Q, 8)
    torch.cuda.synchronize()
    tree.close()
    torch.cuda.empty_cache()
    room = PEAK[(dim, split)] * N + (512 << 20)
    hold = []
    for _ in range(4):  # (what the runtime frees late is taken as well)
        more = torch.cuda.mem_get_info()[0] - room
        if more > 32 << 20:
            hold.append(torch.empty(more, dtype=torch.uint8, device="cuda:0"))
    print(f"[gpu] short memory D={dim} split={split}: {torch.cuda.mem_get_info()[0] >> 20} MB free", flush=True)
    try:
        tree = kd.kd_build(P, split=split)
        assert np.array_equal(tree.order(), order)
        i, d = kd.kd_knn(tree, Q, 8)
        assert torch.equal(i, wi) and torch.equal(d, wd)
        tree.close()
    finally:
        torch.cuda.synchronize()
        del hold
        torch.cuda.empty_cache()
