"""gs_bin_sort on made-up footprints against numpy's stable sort by (tile, depth, record): exact.
Both orders of work (by tile, depth first: the pair capacity decides) at the edges of their
parts: records per work-group, digits of the tile id, footprints left to a wave or a work-group,
lists of one wave, of one work-group and of one and two merges, equal depths, too few pairs."""
import numpy as np
import pytest
import torch

from paper_2404_01133_amd import gs

pytestmark = pytest.mark.gpu


def _expected(view, i0, i1, j0, j1, depth, W, H):
    tx, ty = (W + 15) // 16, (H + 15) // 16
    a, b, c, d = i0 // 16, i1 // 16, j0 // 16, j1 // 16
    w, h = b - a + 1, d - c + 1
    per = w * h
    rec = np.repeat(np.arange(len(view)), per)
    q = np.arange(per.sum()) - np.repeat(np.cumsum(per) - per, per)
    tile = view[rec] * (tx * ty) + (c[rec] + q // w[rec]) * tx + a[rec] + q % w[rec]
    order = np.lexsort((rec, depth[rec], tile))
    return per, tile[order], rec[order], tx * ty


def _check(n, W, H, V, extent, depths, cap_factor, hot=0, culled=0.3, seed=0):
    rng = np.random.default_rng(seed)
    view = rng.integers(0, V, n)
    i0, j0 = rng.integers(0, W, n), rng.integers(0, H, n)
    i1 = np.minimum(W - 1, i0 + rng.integers(0, extent, n))
    j1 = np.minimum(H - 1, j0 + rng.integers(0, extent, n))
    if hot:  # the first records all in tile 0 of view 0
        view[:hot] = i0[:hot] = i1[:hot] = j0[:hot] = j1[:hot] = 0
    depth = rng.choice(np.float32(rng.uniform(0.2, 900.0, depths)), n).view(np.uint32)
    vis = rng.random(n) >= culled
    vis[:hot] = True
    ids = np.nonzero(vis)[0]
    per, tile, rec, tiles_per_view = _expected(view[ids], i0[ids], i1[ids], j0[ids], j1[ids], depth[ids], W, H)
    rec = ids[rec]
    words = rng.integers(0, 1 << 32, (n, 12), dtype=np.uint64).astype(np.uint32)  # culled records are not written
    words[ids, 1] = view[ids]
    words[ids, 2] = i0[ids] | ((i1 - i0)[ids] << 16)
    words[ids, 3] = j0[ids] | ((j1 - j0)[ids] << 16)
    touched = np.zeros(n, np.int32)
    touched[ids] = per
    m = len(rec)
    cap = max(1, int(np.ceil(cap_factor * m)))
    tiles = tiles_per_view * V
    dev = lambda x: torch.from_numpy(np.ascontiguousarray(x).view(np.int32)).cuda()
    t = gs.tuning_struct()
    counts = torch.zeros(gs.GS_COUNT_SLOTS, dtype=torch.int64, device="cuda")
    counts[0] = n
    rc = n + 5
    pad = lambda x: torch.cat([x, torch.zeros((5,) + tuple(x.shape[1:]), dtype=x.dtype, device="cuda")])
    pt, pr = (torch.full((cap,), -1, dtype=torch.int32, device="cuda") for _ in range(2))
    ranges = torch.empty((tiles, 2), dtype=torch.int32, device="cuda")
    ws = torch.empty(gs.workspace_bytes(gs.GS_WS_BIN_SORT, rc, cap, V, W, H, t), dtype=torch.uint8, device="cuda")
    args = (pad(dev(words)), pad(dev(np.where(vis, depth, np.uint32(0xFFFFFFFF)))), pad(dev(touched)))
    for _ in range(2):  # the second call finds the first one's workspace
        gs.bin_sort(*args, V, W, H, t, rc, cap, pt, pr, ranges, counts, ws)
        c = counts.cpu().numpy()
        assert (c[1], c[2], c[3]) == (len(ids), m, 0 if m <= cap else gs.GS_FLAG_PAIRS)
        if m > cap:
            assert int(pr.min()) >= 0 and int(pr.max()) < n  # dropped pairs leave no stale ones
            counts[3] = 0
            continue
        np.testing.assert_array_equal(pt.cpu().numpy()[:m].view(np.uint32), tile)
        np.testing.assert_array_equal(pr.cpu().numpy()[:m].view(np.uint32), rec)
        want = np.stack([np.searchsorted(tile, np.arange(tiles)), np.searchsorted(tile, np.arange(tiles), "right")], 1)
        got = ranges.cpu().numpy()
        full = want[:, 1] > want[:, 0]
        np.testing.assert_array_equal(got[full], want[full])
        assert np.all(got[~full, 0] == got[~full, 1])


# cap_factor 1 gives lists by tile where the means allow it, 40 depth first (more than 4 pairs a record
# and 1M pairs, or 512 a tile)
@pytest.mark.parametrize("cap_factor", [1, 40])
@pytest.mark.parametrize("n,W,H,V,extent,depths", [
    (1, 16, 16, 1, 1, 1),           # one tile: no tile digits
    (1500, 16, 16, 1, 3, 40),       # one list of about 1050
    (63, 200, 100, 3, 20, 5), (4097, 256, 256, 1, 40, 100), (16385, 700, 500, 2, 30, 3),
    (65537, 1920, 1080, 1, 20, 1 << 20), (131073, 1024, 1024, 1, 3, 1), (600_000, 1600, 900, 2, 12, 1 << 20),
    (5000, 8192, 4096, 2, 60, 100),      # 18 bits of tile ids, two digits of 9
    (3000, 2000, 1000, 1, 1400, 1000),   # footprints of up to 5500 tiles
])
def test_binning_equals_a_stable_sort(n, W, H, V, extent, depths, cap_factor):
    _check(n, W, H, V, extent, depths, cap_factor, seed=n)


@pytest.mark.parametrize("hot,depths", [(1024, 7), (1025, 7), (2048, 1), (2049, 1 << 20), (4097, 50), (8193, 1 << 20),
                                        (16384, 1), (16385, 100), (40_000, 1 << 20)])
def test_long_lists(hot, depths):
    _check(hot + 60_000, 600, 500, 1, 4, depths, 1, hot=hot, seed=hot)


def test_list_of_two_merges():
    _check(4_250_000, 640, 640, 1, 2, 1 << 22, 1, hot=4_200_000, culled=0.0)


@pytest.mark.parametrize("n,cap_factor", [(20_000, 0.5), (20_000, 0.999), (600_000, 0.7)])
def test_too_few_pairs(n, cap_factor):
    _check(n, 640, 360, 2, 30, 1 << 20, cap_factor)
