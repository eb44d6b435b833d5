"""Tile lists beyond one work-group's sort: gs_bin_sort by tile (few pairs per record: nearly all of them in one
tile, as in a view from far away) against depth first on the same records.  Same pairs, and the time of a sort
that is linear in the list's length."""
import numpy as np
import pytest
import torch

from paper_2404_01133_amd import gs
from test_gpu_binning_routes import capacity

pytestmark = pytest.mark.gpu

W = H = 640
TILES = 1600


class _Case:
    def __init__(self, n, depths, seed):
        """n records of one tile each, a hundredth of them anywhere, the others in tile 0."""
        g = torch.Generator(device="cuda").manual_seed(seed)
        draw = lambda hi: torch.randint(0, hi, (n,), generator=g, device="cuda")
        apart = draw(100) == 0
        self.n = n
        self.tile = torch.where(apart, draw(TILES), 0)
        values = (torch.rand(depths, generator=g, device="cuda") * 900 + 0.2).view(torch.int32)
        self.keys = values[draw(depths)].contiguous()
        self.records = torch.zeros((n, 12), dtype=torch.int32, device="cuda")
        self.records[:, 2] = self.tile % (W // 16) * 16
        self.records[:, 3] = self.tile // (W // 16) * 16
        self.touched = torch.ones(n, dtype=torch.int32, device="cuda")

    def run(self, route):
        pc = capacity(route, self.n, self.n, TILES)
        t = gs.tuning_struct()
        counts = torch.zeros(gs.GS_COUNT_SLOTS, dtype=torch.int64, device="cuda")
        counts[0] = self.n
        pt, pr = (torch.full((pc,), -1, dtype=torch.int32, device="cuda") for _ in range(2))
        ranges = torch.empty((TILES, 2), dtype=torch.int32, device="cuda")
        ws = torch.empty(gs.workspace_bytes(gs.GS_WS_BIN_SORT, self.n, pc, 1, W, H, t), dtype=torch.uint8,
                         device="cuda")

        def go():
            gs.bin_sort(self.records, self.keys, self.touched, 1, W, H, t, self.n, pc, pt, pr, ranges, counts, ws)
        go()
        assert counts.tolist()[1:4] == [self.n, self.n, 0]
        return go, pt[:self.n], pr[:self.n], ranges


@pytest.mark.parametrize("n,depths", [(20_000, 1), (34_000, 1), (50_000, 3), (200_000, 1 << 20), (1_000_000, 7),
                                      (4_300_000, 1 << 22), (4_500_000, 2)])
def test_long_lists_equal_depth_first(n, depths):
    c = _Case(n, depths, n)
    _, *a = c.run("tile")
    _, *b = c.run("depth")
    for x, y in zip(a, b):
        assert torch.equal(x, y)


@pytest.mark.parametrize("n", [300_000, 2_000_000])
def test_long_lists_cost_no_more_than_the_depth_order(n):
    """By tile, a list is read and written three times more than depth first reads the records, in as many
    passes over LDS: at most three times its time.  (Searching every run for every entry: 13 times for 2M.)"""
    c = _Case(n, 1 << 22, n)
    best = {}
    for route in ("tile", "depth"):
        go = c.run(route)[0]
        a, b = (torch.cuda.Event(enable_timing=True) for _ in range(2))
        for _ in range(5):
            a.record()
            go()
            b.record()
            b.synchronize()
            best[route] = min(best.get(route, 1e9), a.elapsed_time(b))
    print("case:", n, best, flush=True)
    assert best["tile"] <= 3.0 * best["depth"]
