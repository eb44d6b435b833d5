"""Scene set-up kernels at the edges of their searches and orders: MAD boxes of
degenerate blocks against the oracle, gathers against plain indexing (both exact)."""
import numpy as np
import pytest
import torch

from oracle import lod as olod
from paper_2404_01133_amd import gs, render

pytestmark = pytest.mark.gpu


def _mad_blocks():
    rng = np.random.default_rng(5)
    return {
        "one": np.array([3.25]), "two": np.array([1.0, -2.0]), "equal": np.full(9000, -7.5),
        "zeros": np.array([0.0, -0.0] * 3000), "quantised": np.round(rng.normal(size=50_000) * 4) / 4,
        "uniform": rng.uniform(-600, 600, size=70_001), "tiny": rng.normal(size=4097) * 1e-38,
        # most centres at one point: the median deviation lies far below the largest
        "spike": np.concatenate([np.full(30_000, 0.125), rng.normal(size=29_000) * 1e3]),
        "near": np.concatenate([1.0 + rng.uniform(0, 1e-6, size=20_000), [1e6, -1e6]]),
        "wide": np.exp(rng.uniform(-60, 60, size=30_000)) * rng.choice([-1, 1], size=30_000),
    }


def test_mad_boxes_of_degenerate_blocks():
    blocks = _mad_blocks()
    cnt = np.array([0] + [len(v) for v in blocks.values()], np.int64)
    off = np.cumsum(cnt) - cnt
    means = np.concatenate(list(blocks.values())).astype(np.float32)
    means = np.stack([means, -means[::-1], np.roll(means, 1)])  # the other axes mix the blocks
    n = means.shape[1]
    t = torch.from_numpy(means).cuda()
    one = torch.ones(n, device="cuda")
    scene = render.DeviceScene([render.DeviceLevel(t, torch.ones(3, n, device="cuda"), torch.ones(4, n, device="cuda"),
                                                   one, torch.ones(1, 3, n, device="cuda"))],
                               off[:, None], cnt[:, None])
    lo, hi = (x.cpu().numpy() for x in scene.compute_bounds(4.0))
    assert np.all(np.isposinf(lo[0])) and np.all(np.isneginf(hi[0]))
    for b, name in enumerate(blocks, start=1):
        want = olod.mad_bounds(means[:, off[b]:off[b] + cnt[b]], 4.0)
        np.testing.assert_array_equal(lo[b], want[0], err_msg=name)
        np.testing.assert_array_equal(hi[b], want[1], err_msg=name)


@pytest.mark.parametrize("n,n_src,planes,order", [
    (1, 1, 1, "random"), (511, 700, 4, "random"), (262_143, 262_143, 4, "blocks"), (262_144, 262_144, 1, "blocks"),
    (262_145, 300_001, 9, "random"), (400_003, 400_003, 1, "reversed"), (300_000, 5, 1, "random"),
    (524_801, 524_801, 4, "blocks")])
def test_gather_is_exact(n, n_src, planes, order):
    rng = np.random.default_rng(n)
    if order == "blocks":  # ascending inside each of 37 groups of uneven size
        perm = np.argsort(rng.integers(0, 37, size=n_src) ** 2 // 37, kind="stable")[:n]
    elif order == "reversed":
        perm = np.arange(n)[::-1]
    else:
        perm = rng.integers(0, n_src, size=n)
    g = torch.Generator(device="cuda").manual_seed(n)
    shapes = ((3,), (3,), (4,), (), (planes, 3))
    src = [torch.rand((*s, n_src), generator=g, device="cuda") for s in shapes]
    dst = [torch.full((*s, n), -1.0, device="cuda") for s in shapes]
    p = torch.from_numpy(np.ascontiguousarray(perm, np.int64)).cuda()
    gs.gather_gaussians(gs.gaussians_struct(*src), p.to(torch.int32), n, gs.grads_struct(*dst))
    for a, b in zip(src, dst):
        assert torch.equal(a.index_select(-1, p), b), (n, tuple(a.shape))
