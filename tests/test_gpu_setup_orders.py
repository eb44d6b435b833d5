"""gs_gather_gaussians on both sides of the size from which it orders its tiles by source (2^19), against
plain indexing: permutations without runs, descending, repeated indices, sources larger, smaller and much
smaller than the output, every number of SH planes.  Exact."""
import numpy as np
import pytest
import torch

from paper_2404_01133_amd import gs

pytestmark = pytest.mark.gpu

ORDERED = 1 << 19


def _perm(order, n, n_src, rng):
    if order == "blocks":  # ascending inside each of 37 groups of uneven size
        return np.argsort(rng.integers(0, 37, size=n_src) ** 2 // 37, kind="stable")[:n]
    if order == "sparse":  # as many groups as a tile has places for: nearly every index beyond the window
        return np.argsort(rng.integers(0, n_src // 64, size=n_src), kind="stable")[:n]
    if order == "reversed":
        return np.arange(n_src)[::-1][:n]
    if order == "identity":
        return np.arange(n)
    if order == "last":
        return np.full(n, n_src - 1)
    return rng.integers(0, n_src, size=n)


@pytest.mark.parametrize("n,n_src,planes,order", [
    (ORDERED - 1, ORDERED - 1, 4, "blocks"), (ORDERED, ORDERED, 1, "blocks"), (ORDERED + 1, ORDERED + 1, 16, "blocks"),
    (ORDERED, ORDERED, 4, "random"), (ORDERED + 1, 1_200_007, 9, "random"), (700_001, 300_001, 16, "random"),
    (ORDERED + 63, 5, 1, "random"), (ORDERED + 64, 1, 4, "last"), (600_003, 600_003, 9, "reversed"),
    (600_000, 900_001, 16, "sparse"), (ORDERED + 65, ORDERED + 65, 1, "identity"), (ORDERED + 2, 3_000_000, 4, "last")])
def test_ordered_gather_is_exact(n, n_src, planes, order):
    rng = np.random.default_rng(n + planes)
    perm = _perm(order, n, n_src, rng)
    assert len(perm) == n and 0 <= perm.min() and perm.max() < n_src
    g = torch.Generator(device="cuda").manual_seed(n)
    shapes = ((3,), (3,), (4,), (), (planes, 3))
    src = [torch.rand((*s, n_src), generator=g, device="cuda") for s in shapes]
    guard = 1024  # words behind every array that have to stay as they are
    size = [int(np.prod(s)) * n for s in shapes]
    buf = [torch.full((k + guard,), -1.0, device="cuda") for k in size]
    dst = [b[:k].view(*s, n) for b, k, s in zip(buf, size, shapes)]
    p = torch.from_numpy(np.ascontiguousarray(perm, np.int64)).cuda()
    for _ in range(2):  # the second call finds the first one's results where it keeps its order
        gs.gather_gaussians(gs.gaussians_struct(*src), p.to(torch.int32), n, gs.grads_struct(*dst))
        for a, b, full in zip(src, dst, buf):
            assert torch.equal(a.index_select(-1, p), b), (n, tuple(a.shape))
            assert bool((full[b.numel():] == -1.0).all())
