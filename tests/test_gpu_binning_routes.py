"""gs_bin_sort in both orders of work (by tile, depth first) where test_gpu_binning's sizes take only one of
them: a single record, a few, footprints of a work-group each in record order, with enough pairs and too few.
Against numpy's stable sort by (tile, depth, record), exact; the order of work is computed here and asserted."""
import numpy as np
import pytest
import torch

from paper_2404_01133_amd import gs
from test_gpu_binning import _expected

pytestmark = pytest.mark.gpu


def by_tile(rc, pc, tiles):
    few = pc <= 4 * rc
    return pc <= (4096 if few else 512) * tiles and (few or pc <= 1 << 20)


def capacity(route, rc, m, tiles):
    """A pair capacity of at least m for which the binning takes `route`."""
    pc = max(m, 1) if route == "tile" else max(m, 4 * rc + 1, min(512 * tiles, 1 << 20) + 1)
    assert by_tile(rc, pc, tiles) == (route == "tile")
    return pc


def records(n, W, H, V, extent, depths, culled, seed):
    """Projected records (words, depth keys, tiles touched) and their sorted pairs."""
    rng = np.random.default_rng(seed)
    view = rng.integers(0, V, n)
    i0, j0 = rng.integers(0, W, n), rng.integers(0, H, n)
    i1 = np.minimum(W - 1, i0 + rng.integers(0, extent, n))
    j1 = np.minimum(H - 1, j0 + rng.integers(0, extent, n))
    depth = rng.choice(np.float32(rng.uniform(0.2, 900.0, depths)), n).view(np.uint32)
    ids = np.nonzero(rng.random(n) >= culled)[0]
    per, tile, rec, tiles_per_view = _expected(view[ids], i0[ids], i1[ids], j0[ids], j1[ids], depth[ids], W, H)
    words = np.zeros((n, 12), np.uint32)
    words[ids, 1] = view[ids]
    words[ids, 2] = i0[ids] | ((i1 - i0)[ids] << 16)
    words[ids, 3] = j0[ids] | ((j1 - j0)[ids] << 16)
    touched = np.zeros(n, np.int32)
    touched[ids] = per
    keys = np.full(n, 0xFFFFFFFF, np.uint32)
    keys[ids] = depth[ids]
    return words, keys, touched, tile, ids[rec], tiles_per_view * V


def bin_sort(words, keys, touched, V, W, H, tiles, rc, cap):
    dev = lambda x: torch.from_numpy(np.ascontiguousarray(x).view(np.int32)).cuda()
    t = gs.tuning_struct()
    counts = torch.zeros(gs.GS_COUNT_SLOTS, dtype=torch.int64, device="cuda")
    counts[0] = len(keys)
    pt, pr = (torch.full((cap,), -1, dtype=torch.int32, device="cuda") for _ in range(2))
    ranges = torch.empty((tiles, 2), dtype=torch.int32, device="cuda")
    ws = torch.empty(gs.workspace_bytes(gs.GS_WS_BIN_SORT, rc, cap, V, W, H, t), dtype=torch.uint8, device="cuda")
    gs.bin_sort(dev(words), dev(keys), dev(touched), V, W, H, t, rc, cap, pt, pr, ranges, counts, ws)
    return counts.cpu().numpy(), *(x.cpu().numpy().view(np.uint32) for x in (pt, pr, ranges))


@pytest.mark.parametrize("route", ["tile", "depth"])
@pytest.mark.parametrize("n,W,H,V,extent,depths,culled", [
    (1, 16, 16, 1, 1, 1, 0.0), (1, 300, 200, 2, 90, 1, 0.0), (2, 16, 16, 1, 16, 1, 0.0), (63, 200, 100, 3, 20, 5, 0.3),
    (300, 2000, 1000, 1, 1400, 100, 0.3),  # footprints of up to 5500 tiles
])
def test_small_inputs_and_large_footprints(n, W, H, V, extent, depths, culled, route):
    words, keys, touched, tile, rec, tiles = records(n, W, H, V, extent, depths, culled, seed=n)
    m = len(rec)
    assert m >= n * (1 - culled) / 2 and (n != 300 or touched.max() > 512)
    counts, pt, pr, ranges = bin_sort(words, keys, touched, V, W, H, tiles, n, capacity(route, n, m, tiles))
    assert tuple(counts[1:4]) == ((touched > 0).sum(), m, 0)
    np.testing.assert_array_equal(pt[:m], tile)
    np.testing.assert_array_equal(pr[:m], rec)
    for side in ("left", "right"):
        full = np.isin(np.arange(tiles), tile)
        np.testing.assert_array_equal(ranges[full, int(side == "right")],
                                      np.searchsorted(tile, np.nonzero(full)[0], side))
    assert np.all(ranges[~full, 0] == ranges[~full, 1])


@pytest.mark.parametrize("part", [0.6, 0.999])
def test_large_footprints_with_too_few_pairs(part):
    words, keys, touched, tile, rec, tiles = records(300, 2000, 1000, 1, 1400, 100, 0.3, seed=300)
    m, cap = len(rec), int(part * len(rec))
    assert by_tile(300, cap, tiles) and touched.max() > 512
    counts, pt, pr, ranges = bin_sort(words, keys, touched, 1, 2000, 1000, tiles, 300, cap)
    assert tuple(counts[1:4]) == ((touched > 0).sum(), m, gs.GS_FLAG_PAIRS)
    # the kept pairs are the first in record order, row by row: grouped by tile, every list in order of depth
    order = np.lexsort((tile, rec))
    kept = order[:cap]
    kept = kept[np.lexsort((rec[kept], keys[rec[kept]], tile[kept]))]
    np.testing.assert_array_equal(pt, tile[kept])
    np.testing.assert_array_equal(pr, rec[kept])
