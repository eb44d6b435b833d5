"""The work this framework is used for, as cases that can be timed and checked.

A case names one call of the public Python entry points (paper_2404_01133_amd.render,
.gs and .assignment) with its sizes and options.  Kinds:

  raster   render.rasterize of one Gaussian set (every Gaussian, LoD off): a forward
           render, or a training step that returns the image and all gradients
  lod      render.render_frame of a city split into blocks with three nested detail
           levels: block-wise selection with the chunk refinement, or the point-wise
           baseline; coarse levels in FP32 or in binary16 with fewer SH bands; with
           train, the gradients of every level too (render.backward_frame)
  setup    what a scene goes through once: block partition of an unordered cloud in
           contracted space, gather into block order, MAD boxes, chunk boxes
  assign   assignment.assign_poses: leave-one-block-out renders and their SSIM

Inputs are drawn on the GPU from the seed with the distributions of the repository's
synthetic scenes (log-scales N(-3, 0.5), unit quaternions, opacity sigmoid(N(0, 1)),
SH N(0, 0.3); city with 40 % ground, buildings on 40 m lots, 0.5 % floaters, Morton
order inside a block).
"""
from __future__ import annotations

import math
from types import SimpleNamespace

import numpy as np
import torch

DEV = "cuda"
THRESHOLDS = (200.0, 500.0)   # distance intervals of the three levels, metres
FRACTIONS = (0.30, 0.50, 1.00)  # share of the finest level that each level keeps
COARSE_SCALE = 1.3
CITY_DENSITY = 20e6 / 1.5e6   # finest Gaussians per square metre
SH_BANDS = (1, 2, 3)          # bands stored per level when coarse levels are reduced
Z_TOP = 160.0


# ---------------------------------------------------------------------------
# the cases
# ---------------------------------------------------------------------------
def _raster(name, n, width, height, views=1, train=True, shape="cube", sh_degree=3, bg=0.0, keep=True, shared=False):
    return dict(name=name, kind="raster", n=n, width=width, height=height, views=views, train=train, shape=shape,
                sh_degree=sh_degree, bg=bg, keep=keep, shared=shared)


def _lod(name, n, grid, width, height, views, mode="block", half=False, train=False, check=False, cam_height=0.0,
         pitch=0.0):
    return dict(name=name, kind="lod", n=n, grid=grid, width=width, height=height, views=views, mode=mode, half=half,
                train=train, check=check, cam_height=cam_height, pitch=pitch)


def listed():
    return [
        # a preview of a small set: launches and host latency count
        _raster("plain_4k_view", 4096, 256, 256, train=False),
        # one optimiser step on the same set (a unit test, a toy fit)
        _raster("plain_4k_train", 4096, 256, 256),
        # the quick call with no frame kept: odd sizes, two SH bands, a background, two views
        _raster("plain_ragged_train", 70_001, 611, 397, views=2, sh_degree=2, bg=0.25, keep=False),
        # one training view of a mid-sized aerial capture
        _raster("plain_1m_train", 1_000_000, 1920, 1080, shape="box"),
        # batched training views of one 2M-Gaussian block: the largest step
        _raster("block_16_views_train", 2_000_000, 1600, 900, views=16, shape="block", shared=True),
        # interactive viewing of the 20M city: one view, checked, at the middle height looking ahead
        _lod("city_view", 20_000_000, 8, 1600, 900, 1, check=True, cam_height=150.0, pitch=-45.0),
        # serving: eight views per call (all heights and pitches), nothing read back
        _lod("city_8_views", 20_000_000, 8, 1600, 900, 8),
        # the same with binary16 coarse levels on a mid-sized city
        _lod("city_half_views", 6_000_000, 5, 1280, 720, 4, half=True),
        # fine-tuning over several LoD views whose blocks take different levels
        _lod("city_train", 3_000_000, 4, 1280, 720, 4, train=True),
        # the point-wise selection baseline, one view
        _lod("city_points_view", 6_000_000, 5, 1600, 900, 1, mode="points", check=True, cam_height=150.0, pitch=-45.0),
        # a new scene of 5M Gaussians brought into blocks
        dict(name="scene_setup", kind="setup", n=5_000_000, grid=6),
        # training-data assignment of a few poses to the blocks of a coarse prior
        dict(name="assign_poses", kind="assign", n=1_000_000, grid=6, poses=6, width=960, height=540),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["raster", "raster", "raster", "lod", "lod", "lod", "setup", "assign"])
    if kind == "raster":
        shape = rng.choice(["cube", "box", "block"])
        views = rng.choice([1, 1, 2, 3, 5, 8])
        c = _raster("", _log(rng, 3000, 1_000_000 if views < 3 else 400_000), _log(rng, 200, 1600),
                    _log(rng, 150, 900), views=views, train=rng.random() < 0.75, shape=shape,
                    sh_degree=rng.choice([0, 1, 2, 3, 3, 3]), bg=rng.choice([0.0, 0.0, 0.5]),
                    keep=rng.random() < 0.8, shared=views > 1 and rng.random() < 0.7)
    elif kind == "lod":
        train = rng.random() < 0.35
        mode = "points" if rng.random() < 0.2 else "block"
        n = _log(rng, 300_000, 4_000_000 if train else 16_000_000)
        c = _lod("", n, max(2, min(8, int(math.sqrt(n / 312_500)) + rng.randrange(2))), _log(rng, 320, 1600),
                 _log(rng, 200, 900), rng.randrange(1, 5 if train or mode == "points" else 9), mode=mode,
                 half=rng.random() < 0.3, train=train, check=rng.random() < 0.3)
    elif kind == "setup":
        c = dict(kind="setup", n=_log(rng, 100_000, 8_000_000), grid=rng.randrange(2, 10))
    else:
        c = dict(kind="assign", n=_log(rng, 100_000, 1_000_000), grid=rng.randrange(3, 7), poses=rng.randrange(1, 7),
                 width=_log(rng, 300, 960), height=_log(rng, 200, 540))
    c.pop("name", None)
    return c


# ---------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------
def _gen(seed):
    return torch.Generator(device=DEV).manual_seed(int(seed))


def _look(center, yaw, pitch, width, height, fov_deg=60.0, znear=0.2):
    """World -> camera pose at `center` (camera axes x right, y down, z forward; world z up)."""
    fwd = np.array([math.cos(pitch) * math.cos(yaw), math.cos(pitch) * math.sin(yaw), math.sin(pitch)])
    right = np.array([math.sin(yaw), -math.cos(yaw), 0.0])
    down = np.cross(fwd, right)
    down /= np.linalg.norm(down)
    R = np.stack([right, down, fwd])
    f = (0.5 * width) / math.tan(math.radians(0.5 * fov_deg))
    return SimpleNamespace(R=R, t=-R @ np.asarray(center, np.float64), fx=f, fy=f, cx=0.5 * width, cy=0.5 * height,
                           znear=znear, width=int(width), height=int(height))


def _attributes(n, g):
    scales = torch.exp(torch.randn((3, n), generator=g, device=DEV) * 0.5 - 3.0)
    quats = torch.randn((4, n), generator=g, device=DEV)
    quats /= quats.norm(dim=0, keepdim=True)
    opac = torch.sigmoid(torch.randn(n, generator=g, device=DEV))
    sh = torch.randn((16, 3, n), generator=g, device=DEV) * 0.3
    return scales, quats, opac, sh


def _city_points(n, side, g, lot=40.0, footprint=25.0):
    """Centres of a city over [-side/2, side/2]^2 (float64 [3, n])."""
    def uni(k):
        return torch.rand(k, generator=g, device=DEV, dtype=torch.float64)

    n_ground, n_float = int(round(0.40 * n)), int(round(0.005 * n))
    n_bld = n - n_ground - n_float
    nl = max(1, int(side // lot))
    h = torch.exp(math.log(20.0) + 0.6 * torch.randn(nl * nl, generator=g, device=DEV, dtype=torch.float64))
    h = h.clamp(5.0, 150.0)
    at = torch.arange(nl * nl, device=DEV)
    bx0 = -0.5 * side + lot * (at // nl) + 0.5 * (lot - footprint)
    by0 = -0.5 * side + lot * (at % nl) + 0.5 * (lot - footprint)
    cdf = torch.cumsum(4.0 * footprint * h + footprint * footprint, 0)
    b = torch.searchsorted(cdf, uni(n_bld) * cdf[-1], right=True).clamp(max=nl * nl - 1)
    s, t, face = uni(n_bld) * footprint, uni(n_bld), uni(n_bld)
    hb = h[b]
    roof = face * (4.0 * footprint * hb + footprint * footprint) < footprint * footprint
    wall = (uni(n_bld) * 4).long()
    fx = torch.where(wall == 1, footprint, torch.where(wall == 3, 0.0, s))
    fy = torch.where(wall == 0, 0.0, torch.where(wall == 2, footprint, s))
    px = bx0[b] + torch.where(roof, s, fx)
    py = by0[b] + torch.where(roof, t * footprint, fy)
    pz = torch.where(roof, hb, hb * t)
    flat = torch.stack([(uni(n_ground + n_float) - 0.5) * side, (uni(n_ground + n_float) - 0.5) * side])
    z = torch.cat([uni(n_ground) * 0.5, uni(n_float) * 300.0])
    return torch.cat([torch.stack([px, py, pz]), torch.cat([flat, z[None]])], dim=1)


def _spread(v):
    v = v & 0x3FF
    v = (v | (v << 16)) & 0x030000FF
    v = (v | (v << 8)) & 0x0300F00F
    v = (v | (v << 4)) & 0x030C30C3
    return (v | (v << 2)) & 0x09249249


def _blocks_in_order(means, side, grid):
    """(order, block ids in that order, cells): by block, Morton order inside a block."""
    cell = side / grid
    x0 = -0.5 * side
    bx = ((means[0] - x0) / cell).floor().clamp(0, grid - 1).long()
    by = ((means[1] - x0) / cell).floor().clamp(0, grid - 1).long()
    block = by * grid + bx
    q = [(a * 1024.0).clamp(0, 1023).long() for a in ((means[0] - (x0 + bx * cell)) / cell,
                                                      (means[1] - (x0 + by * cell)) / cell, means[2] / Z_TOP)]
    code = _spread(q[0]) | (_spread(q[1]) << 1) | (_spread(q[2]) << 2)
    order = torch.argsort((block << 30) | code, stable=True)
    k = np.arange(grid * grid)
    cx, cy = x0 + cell * (k % grid), x0 + cell * (k // grid)
    return order, block[order], np.stack([cx, cx + cell, cy, cy + cell], axis=1)


def _single_set(case, g):
    """One Gaussian set and its cameras for the raster kind."""
    n, W, H, V = case["n"], case["width"], case["height"], case["views"]
    rng = np.random.default_rng(int(torch.randint(1 << 30, (1,), generator=g, device=DEV)))
    if case["shape"] == "cube":
        means = torch.rand((3, n), generator=g, device=DEV) * 2.0 - 1.0
        cams = [_look((0.0, -3.0 - 0.2 * k, 0.3 * k), math.pi / 2 + 0.05 * k, -0.1 * k, W, H) for k in range(V)]
    elif case["shape"] == "box":  # 200 x 200 x 40 m seen from 60 m up, 45 degrees down
        means = torch.rand((3, n), generator=g, device=DEV) * torch.tensor([[200.0], [200.0], [40.0]], device=DEV)
        means -= torch.tensor([[100.0], [100.0], [0.0]], device=DEV)
        cams = [_look((10.0 * k, -100.0 + 5.0 * k, 60.0), math.pi / 2 + 0.1 * k, -math.pi / 4, W, H)
                for k in range(V)]
    else:  # one city block, orbited
        side, r = 153.1, 60.0
        means = _city_points(n, side, g)
        means = means[:, _blocks_in_order(means, side, 1)[0]].float().contiguous()
        a0 = rng.uniform(0.0, 2 * math.pi)
        cams = []
        for k in range(V):
            a = a0 + 2 * math.pi * k / V
            cams.append(_look((r * math.cos(a), r * math.sin(a), r), a + math.pi, -math.pi / 4, W, H))
    return (means, *_attributes(n, g)), cams


def _city(case, g):
    """Levels (coarsest first, FP32 tuples), block table and cameras for the lod kind."""
    n, grid = case["n"], case["grid"]
    side = math.sqrt(n / CITY_DENSITY)
    means = _city_points(n, side, g)
    order, block, cells = _blocks_in_order(means, side, grid)
    means = means[:, order].float().contiguous()
    fine = (means, *_attributes(n, g))
    shuffled = torch.randperm(n, generator=g, device=DEV)
    levels, counts = [], []
    for f in FRACTIONS:
        if f >= 1.0:
            levels.append(fine)
            counts.append(torch.bincount(block, minlength=grid * grid))
            continue
        idx = torch.sort(shuffled[:int(f * n)]).values  # nested: a level holds every coarser one's
        m, s, q, o, sh = (t.index_select(t.dim() - 1, idx) for t in fine)
        levels.append((m, s * torch.tensor(COARSE_SCALE, device=DEV), q, o, sh))
        counts.append(torch.bincount(block[idx], minlength=grid * grid))
    lvl_cnt = torch.stack(counts, dim=1).cpu().numpy()
    lvl_off = np.zeros_like(lvl_cnt)
    lvl_off[1:] = np.cumsum(lvl_cnt, axis=0)[:-1]
    rng = np.random.default_rng(int(torch.randint(1 << 30, (1,), generator=g, device=DEV)))
    cams = []
    for k in range(case["views"]):
        x, y = rng.uniform(-0.4 * side, 0.4 * side, size=2)
        height = case["cam_height"] or (50.0, 150.0, 400.0)[k % 3]
        pitch = case["pitch"] or (-90.0, -45.0)[k % 2]
        cams.append(_look((x, y, height), rng.uniform(0.0, 2 * math.pi), math.radians(pitch), case["width"],
                          case["height"]))
    return levels, lvl_off, lvl_cnt, cells, cams


def _cloud(case, g):
    """An unordered cloud wider than its foreground box: (arrays, xy box of the central third)."""
    n = case["n"]
    side = math.sqrt(n / CITY_DENSITY)
    means = _city_points(n, side, g)
    means = means[:, torch.randperm(n, generator=g, device=DEV)].float().contiguous()
    return (means, *_attributes(n, g)), (-side / 6, -side / 6, side / 6, side / 6)


def _assign_cams(case, g):
    side = math.sqrt(case["n"] / (3e6 / 1.5e6))
    rng = np.random.default_rng(int(torch.randint(1 << 30, (1,), generator=g, device=DEV)))
    cams = []
    for k in range(case["poses"]):
        x, y = rng.uniform(-0.4 * side, 0.4 * side, size=2)
        cams.append(_look((x, y, (100.0, 200.0)[k % 2]), rng.uniform(0.0, 2 * math.pi),
                          math.radians((-90.0, -45.0)[(k // 2) % 2]), case["width"], case["height"]))
    return cams, side


def _assign_inputs(case, g):
    """A coarse prior (2 Gaussians per square metre) in a contracted block grid, and poses."""
    cams, side = _assign_cams(case, g)
    means = _city_points(case["n"], side, g).float().contiguous()
    return (means, *_attributes(case["n"], g)), (-side / 6, -side / 6, side / 6, side / 6), cams


# ---------------------------------------------------------------------------
# prepare and run
# ---------------------------------------------------------------------------
def _partitioned(render, gs, arrays, box, grid):
    """The block table of an unordered cloud, on the device (one level)."""
    n = arrays[3].shape[0]
    src = render.DeviceLevel(*arrays)
    perm = torch.empty(n, dtype=torch.int32, device=DEV)
    block_off = torch.empty(grid * grid + 1, dtype=torch.int64, device=DEV)
    cells = torch.empty((grid * grid, 4), dtype=torch.float64, device=DEV)
    ws = torch.empty(gs.partition_workspace_bytes(n), dtype=torch.uint8, device=DEV)
    gs.partition(src.means, n, box, grid, grid, perm, block_off, ws, cells=cells)
    dst = render.DeviceLevel(*(torch.empty_like(t) for t in arrays))
    gs.gather_gaussians(src.struct(), perm, n, gs.grads_struct(dst.means, dst.scales, dst.quats, dst.opac, dst.sh))
    return dst, perm, block_off, cells


def prepare(case, seed):
    from paper_2404_01133_amd import gs, render

    g = _gen(seed)
    s = SimpleNamespace(case=case, gs=gs, render=render)
    W, H = case.get("width"), case.get("height")
    if case["kind"] == "raster":
        params, s.cams = _single_set(case, g)
        s.params = [p.contiguous().requires_grad_(case["train"]) for p in params]
        V, n = case["views"], case["n"]
        s.d_rgb = torch.randn((V, 3, H, W), generator=g, device=DEV) if case["train"] else None
        s.frame = None
        if case["keep"] or case["shared"]:
            flags = gs.GS_TUNE_SHARED_SELECTION if case["shared"] else 0
            s.frame = render.Frame(1, V, W, H, V * n, max(1 << 16, 2 * V * n), gs.tuning_struct(flags=flags),
                                   device=DEV)
    elif case["kind"] == "lod":
        levels, lvl_off, lvl_cnt, cells, cams = _city(case, g)
        s.scene = render.DeviceScene([render.DeviceLevel(*lv) for lv in levels], lvl_off, lvl_cnt, cells=cells,
                                     device=DEV)
        s.scene.compute_bounds(4.0)
        if case["half"]:
            s.scene = s.scene.reduced_precision(SH_BANDS)
        s.cams_dev = gs.cameras_to_device(cams, DEV)
        s.frame = render.Frame(s.scene.n_blocks, case["views"], W, H, 1 << 16, 1 << 16, device=DEV)
        s.mode = render.LOD_POINTWISE if case["mode"] == "points" else gs.GS_LOD_BLOCKWISE
        render.render_frame(s.scene, s.frame, s.cams_dev, s.mode, THRESHOLDS, refine=case["mode"] == "block")
        if case["train"]:
            s.d_rgb = torch.randn((case["views"], 3, H, W), generator=g, device=DEV)
            s.grads = [lv.zeros_like() for lv in s.scene.levels]
    elif case["kind"] == "setup":
        s.arrays, s.box = _cloud(case, g)
    else:
        arrays, box, s.cams = _assign_inputs(case, g)
        lv, perm, off, cells = _partitioned(render, gs, arrays, box, case["grid"])
        cnt = torch.diff(off).cpu().numpy()[:, None]
        s.scene = render.DeviceScene([lv], off[:-1].cpu().numpy()[:, None], cnt, cells=cells.cpu().numpy(),
                                     device=DEV)
        z = lv.means[2]
        s.scene.contraction = torch.tensor([box[0], box[1], float(z.min()), box[2], box[3], float(z.max())],
                                           dtype=torch.float64, device=DEV)
    return s


def run(s):
    case, render = s.case, s.render
    if case["kind"] == "raster":
        bg = (case["bg"],) * 3
        if not case["train"]:
            with torch.no_grad():
                return {"rgb": render.rasterize(*s.params, s.cams, case["sh_degree"], bg, s.frame)}
        rgb = render.rasterize(*s.params, s.cams, case["sh_degree"], bg, s.frame)
        grads = torch.autograd.grad(rgb, s.params, s.d_rgb)
        return {"rgb": rgb.detach(), "grads": list(grads)}
    if case["kind"] == "lod":
        f = s.frame
        render.render_frame(s.scene, f, s.cams_dev, s.mode, THRESHOLDS, check=case["check"],
                            refine=case["mode"] == "block")
        out = {"rgb": f.rgb, "T": f.T}
        if case["train"]:
            for lv in s.grads:
                for t in (lv.means, lv.scales, lv.quats, lv.opac, lv.sh):
                    t.zero_()
            render.backward_frame(s.scene, f, s.cams_dev, s.d_rgb, s.grads)
            out["grads"] = [[lv.means, lv.scales, lv.quats, lv.opac, lv.sh] for lv in s.grads]
        return out
    if case["kind"] == "setup":
        lv, perm, off, cells = _partitioned(render, s.gs, s.arrays, s.box, case["grid"])
        off_host = off.cpu().numpy()
        scene = render.DeviceScene([lv], off_host[:-1, None], np.diff(off_host)[:, None], device=DEV)
        scene.compute_bounds(4.0)
        scene.ensure_chunks()
        # entries past the scene's chunks are not written; the last word of an entry holds an index's bits
        real = (torch.arange(scene.max_chunks, device=DEV) < scene.chunk_off[-1])[:, None]
        chunks = torch.where(real, scene.chunk_bounds.view(torch.int32), 0)
        return {"perm": perm, "off": off, "cells": cells, "level": [lv.means, lv.scales, lv.quats, lv.opac, lv.sh],
                "lo": scene.lo, "hi": scene.hi, "chunk_off": scene.chunk_off,
                "chunks": chunks[:, :7].contiguous().view(torch.float32), "chunk_run": chunks[:, 7]}
    from paper_2404_01133_amd import assignment
    r = assignment.assign_poses(s.scene, s.cams, case["width"], case["height"])
    return {"ssim": r["ssim"], "b": r["b"].astype(np.uint8), "b1": r["b1"].astype(np.uint8),
            "b2": r["b2"].astype(np.uint8)}


# ---------------------------------------------------------------------------
# what a pass cannot do without
# ---------------------------------------------------------------------------
# share of a set that is visible in a view, and entries composited per pixel up to its termination (a
# Gaussian whose footprint holds the pixel), of the kinds of set; counted on the listed cases
_VISIBLE = {"cube": 1.0, "box": 0.12, "block": 0.39}
_EVALS = {"cube": 74.0, "box": 9.3, "block": 25.0}
_CITY_VISIBLE, _CITY_EVALS = 0.33, 9.5  # visible Gaussians of a selected city per pixel; entries per pixel


def work(case):
    n = case["n"]
    if case["kind"] == "setup":
        # centres read for the partition; every attribute read and written; centres read for the boxes;
        # centres and scales for the chunks
        return {"bytes": n * (12.0 + 4.0 + 2 * 236.0 + 12.0 + 24.0), "flops": n * 40.0}
    px = case["width"] * case["height"]
    if case["kind"] == "assign":
        # per pose one full render and about 12 leave-one-out renders of blocks it sees, each compared (SSIM)
        renders = case["poses"] * 13.0
        return {"bytes": renders * (px * 24.0 + 0.1 * n * 236.0), "flops": renders * px * (40.0 * 15 + 3 * 2 * 11 * 10)}
    V = case["views"]
    if case["kind"] == "raster":
        k = 3 * (case["sh_degree"] + 1) ** 2
        vis = _VISIBLE[case["shape"]] * n
        evals = _EVALS[case["shape"]] * px * V
        b = n * 28.0 + vis * (16.0 + 4.0 * k) + px * V * 12.0
        if case["train"]:
            b += px * V * 12.0 + n * (44.0 + 4.0 * k) + vis * 4.0 * (11 + k)
        return {"bytes": b, "flops": evals * (60.0 if case["train"] else 15.0)}
    vis = min(_CITY_VISIBLE * px, 0.3 * n)
    evals = _CITY_EVALS * px * V
    per = 130.0 if case["half"] else 236.0
    b = V * vis * (per + 12.0) + px * V * 16.0
    if case["mode"] == "points":
        b += 1.8 * n * 12.0
    if case["train"]:
        b += px * V * 12.0 + 1.8 * n * 236.0 + V * vis * 236.0
    return {"bytes": b, "flops": evals * (60.0 if case["train"] else 15.0)}


# ---------------------------------------------------------------------------
# the same results in 64 bits, plain torch
# ---------------------------------------------------------------------------
_SH = (0.28209479177387814, 0.4886025119029199, 1.0925484305920792, 0.31539156525252005, 0.5462742152960396,
       0.5900435899266435, 2.890611442640554, 0.4570457994644658, 0.3731763325901154, 1.445305721320277)


def _sh_colour(d, sh, degree):
    """Colour of the real SH series sh [K, 3, n] at unit directions d [3, n]."""
    x, y, z = d
    c0, c1, c2a, c2b, c2c, c3a, c3b, c3c, c3d, c3e = _SH
    basis = [c0 * torch.ones_like(x)]
    if degree > 0:
        basis += [-c1 * y, c1 * z, -c1 * x]
    if degree > 1:
        xx, yy, zz = x * x, y * y, z * z
        basis += [c2a * x * y, -c2a * y * z, c2b * (2 * zz - xx - yy), -c2a * x * z, c2c * (xx - yy)]
    if degree > 2:
        basis += [-c3a * y * (3 * xx - yy), c3b * x * y * z, -c3c * y * (4 * zz - xx - yy),
                  c3d * z * (2 * zz - 3 * xx - 3 * yy), -c3c * x * (4 * zz - xx - yy), c3e * z * (xx - yy),
                  -c3a * x * (xx - 3 * yy)]
    return sum(b[None] * sh[k] for k, b in enumerate(basis))


def _project(p, cam, degree):
    """Screen-space Gaussians of a set p = (means, scales, quats, opac, sh) in FP64 for one camera: values
    [9, k] (u, v, conic, opacity, colour), pixel rectangles, depths and the indices of the k visible ones."""
    m, s, q, o, sh = p
    W, H = cam.width, cam.height
    R = torch.tensor(np.asarray(cam.R), dtype=torch.float64, device=DEV)
    t0 = torch.tensor(np.asarray(cam.t), dtype=torch.float64, device=DEV)
    t = R @ m + t0[:, None]
    tz = t[2]
    ok = (tz > cam.znear) & (o >= 1.0 / 255.0)
    rz = 1.0 / torch.where(ok, tz, torch.ones_like(tz))
    ux, uy = t[0] * rz, t[1] * rz
    u, v = cam.fx * ux + cam.cx, cam.fy * uy + cam.cy
    lx, ly = 1.3 * 0.5 * W / cam.fx, 1.3 * 0.5 * H / cam.fy
    w, x, y, z = q / q.norm(dim=0, keepdim=True)
    rot = torch.stack([torch.stack([1 - 2 * (y * y + z * z), 2 * (x * y - w * z), 2 * (x * z + w * y)]),
                       torch.stack([2 * (x * y + w * z), 1 - 2 * (x * x + z * z), 2 * (y * z - w * x)]),
                       torch.stack([2 * (x * z - w * y), 2 * (y * z + w * x), 1 - 2 * (x * x + y * y)])])
    WL = torch.tensordot(R, rot * s[None], dims=1)
    M0 = cam.fx * rz * (WL[0] - ux.clamp(-lx, lx) * WL[2])
    M1 = cam.fy * rz * (WL[1] - uy.clamp(-ly, ly) * WL[2])
    n0, n1, b = (M0 * M0).sum(0), (M1 * M1).sum(0), (M0 * M1).sum(0)
    a, c = n0 + 0.3, n1 + 0.3
    cross = torch.linalg.cross(M0, M1, dim=0)
    det = (cross * cross).sum(0) + 0.3 * (n0 + n1) + 0.09
    with torch.no_grad():
        r = torch.ceil(3.0 * torch.sqrt(0.5 * (a + c) + torch.sqrt((0.5 * (a - c)) ** 2 + b * b)))
        i0, i1 = torch.ceil(u - r - 0.5).clamp(min=0), torch.floor(u + r - 0.5).clamp(max=W - 1)
        j0, j1 = torch.ceil(v - r - 0.5).clamp(min=0), torch.floor(v + r - 0.5).clamp(max=H - 1)
        ok = torch.nonzero(ok & (i0 <= i1) & (j0 <= j1))[:, 0]
        rect = torch.stack([i0, i1, j0, j1])[:, ok].long()
        depth = tz[ok].float()
    centre = -(R.T @ t0)
    d = m[:, ok] - centre[:, None]
    rgb = (_sh_colour(d / d.norm(dim=0, keepdim=True), sh[:, :, ok], degree) + 0.5).clamp(min=0.0)
    flat = torch.cat([torch.stack([u, v, c / det, -b / det, a / det, o])[:, ok], rgb])
    return flat, rect, depth, ok


def _composite(flat, rect, depth, W, H, bg, d_rgb=None, cells=48_000_000):
    """(rgb [3, H, W], T [H, W]) of the screen-space Gaussians flat [9, n]; with d_rgb, also the
    gradient of sum(d_rgb * rgb) with respect to flat."""
    TS = 16
    tx, ty = (W + TS - 1) // TS, (H + TS - 1) // TS
    order = torch.argsort(depth, stable=True)
    r = rect[:, order] // TS
    nx, cnt = r[1] - r[0] + 1, (r[1] - r[0] + 1) * (r[3] - r[2] + 1)
    rec = torch.repeat_interleave(torch.arange(order.numel(), device=DEV), cnt)
    k = torch.arange(rec.numel(), device=DEV) - (torch.cumsum(cnt, 0) - cnt)[rec]
    tile = (r[2][rec] + k // nx[rec]) * tx + r[0][rec] + k % nx[rec]
    by_tile = torch.argsort(tile, stable=True)
    ids = order[rec[by_tile]]
    length = torch.bincount(tile, minlength=tx * ty)
    first = torch.cumsum(length, 0) - length
    rgb = torch.zeros((3, ty * TS, tx * TS), dtype=torch.float64, device=DEV) + bg
    T = torch.ones((ty * TS, tx * TS), dtype=torch.float64, device=DEV)
    leaf = flat.detach().requires_grad_(d_rgb is not None)
    grad = torch.zeros_like(flat) if d_rgb is not None else None
    if d_rgb is not None:
        d_pad = torch.zeros_like(rgb)
        d_pad[:, :H, :W] = d_rgb
    tiles = torch.argsort(length, descending=True)
    tiles = tiles[length[tiles] > 0]
    lens = length[tiles].cpu().numpy()
    at = 0
    sub = torch.arange(TS * TS, device=DEV)
    while at < len(lens):
        L = int(lens[at])
        m = max(1, min(len(lens) - at, cells // (L * TS * TS)))
        tb = tiles[at:at + m]
        at += m
        slot = torch.arange(L, device=DEV)[None]
        real = slot < length[tb][:, None]
        g = ids[torch.where(real, first[tb][:, None] + slot, 0)]             # [m, L]
        py = (tb // tx)[:, None] * TS + (sub // TS)[None]                    # [m, 256]
        px = (tb % tx)[:, None] * TS + (sub % TS)[None]
        with torch.set_grad_enabled(d_rgb is not None):
            e = leaf[:, g]                                                   # [9, m, L]
            dx = (px + 0.5)[:, :, None] - e[0][:, None]
            dy = (py + 0.5)[:, :, None] - e[1][:, None]
            power = 0.5 * (e[2][:, None] * dx * dx + e[4][:, None] * dy * dy) + e[3][:, None] * dx * dy
            alpha = (e[5][:, None] * torch.exp(-power)).clamp(max=0.99)
            with torch.no_grad():
                ri = rect[:, g][:, :, None]
                use = (real[:, None] & (px[:, :, None] >= ri[0]) & (px[:, :, None] <= ri[1]) &
                       (py[:, :, None] >= ri[2]) & (py[:, :, None] <= ri[3]) & (alpha >= 1.0 / 255.0))
            alpha = torch.where(use, alpha, 0.0)
            T_in = torch.cumprod(1.0 - alpha, dim=2)
            with torch.no_grad():
                keep = T_in >= 1e-4
            T_ex = torch.cat([torch.ones_like(T_in[:, :, :1]), T_in[:, :, :-1]], dim=2)
            weight = torch.where(keep, alpha * T_ex, 0.0)
            T_end = torch.where(keep, T_in, 1.0).amin(dim=2)
            col = torch.matmul(weight, e[6:].permute(1, 2, 0).contiguous()) + bg * T_end[:, :, None]  # [m, 256, 3]
            if d_rgb is not None:
                grad += torch.autograd.grad((col * d_pad[:, py, px].permute(1, 2, 0)).sum(), leaf)[0]
        rgb[:, py, px] = col.detach().permute(2, 0, 1)
        T[py, px] = T_end.detach()
        del e, dx, dy, power, alpha, use, T_in, T_ex, weight, T_end, col, ri, keep
    return rgb[:, :H, :W], T[:H, :W], grad


def _exact_view(p, cam, degree, bg, d_rgb=None):
    """(rgb, T, gradients of p or None) of one view in FP64."""
    if d_rgb is None:
        with torch.no_grad():
            flat, rect, depth, _ = _project(p, cam, degree)
            return (*_composite(flat, rect, depth, cam.width, cam.height, bg)[:2], None)
    leaves = [t.detach().requires_grad_(True) for t in p]
    flat, rect, depth, _ = _project(leaves, cam, degree)
    rgb, T, grad = _composite(flat, rect, depth, cam.width, cam.height, bg, d_rgb)
    return rgb, T, torch.autograd.grad(flat, leaves, grad)


def _lower_median(x):
    return torch.sort(x).values[(x.numel() - 1) // 2]


def _mad_box(pts):
    """Median-absolute-deviation box (4 deviations, clipped to the extremes) of centres [3, n]."""
    lo, hi = [], []
    for x in pts.double():
        med = _lower_median(x)
        dev = 4.0 * _lower_median((x - med).abs())
        lo.append(torch.maximum(x.min(), med - dev))
        hi.append(torch.minimum(x.max(), med + dev))
    return torch.stack(lo), torch.stack(hi)


def _block_level(lo, hi, cell, cam):
    """Level of one block for one camera, -1 if it is not rendered."""
    C = -np.asarray(cam.R).T @ np.asarray(cam.t)
    pts = np.array([[(hi if k & 1 else lo)[0], (hi if k & 2 else lo)[1], (hi if k & 4 else lo)[2]] for k in range(8)])
    d = np.sqrt(((pts - C) ** 2).sum(axis=1).min())
    t = pts @ np.asarray(cam.R).T + np.asarray(cam.t)
    t = t[t[:, 2] > cam.znear]
    seen = cell[0] <= C[0] < cell[1] and cell[2] <= C[1] < cell[3]
    if len(t):
        u, v = cam.fx * t[:, 0] / t[:, 2] + cam.cx, cam.fy * t[:, 1] / t[:, 2] + cam.cy
        seen |= (min(u.max(), cam.width) > max(u.min(), 0.0)) and (min(v.max(), cam.height) > max(v.min(), 0.0))
    return sum(d < th for th in THRESHOLDS) if seen else -1


def _select(case, levels, lvl_off, lvl_cnt, boxes, cells, cam):
    """(level, index) pieces of one view's selection, in record order."""
    if case["mode"] == "points":
        R = torch.tensor(np.asarray(cam.R), dtype=torch.float64, device=DEV)
        t0 = torch.tensor(np.asarray(cam.t), dtype=torch.float64, device=DEV)
        out = []
        for l, lv in enumerate(levels):
            m = lv[0].double()
            d = (m + (R.T @ t0)[:, None]).norm(dim=0)
            t = R @ m + t0[:, None]
            u, v = cam.fx * t[0] / t[2] + cam.cx, cam.fy * t[1] / t[2] + cam.cy
            near = 0.0 if l == 2 else THRESHOLDS[1 - l]
            far = math.inf if l == 0 else THRESHOLDS[2 - l]
            keep = ((d >= near) & (d < far) & (t[2] > cam.znear) & (u > -0.15 * cam.width) & (u < 1.15 * cam.width) &
                    (v > -0.15 * cam.height) & (v < 1.15 * cam.height))
            out.append((l, torch.nonzero(keep)[:, 0]))
        return out
    out = []
    for b, (lo, hi) in enumerate(boxes):
        if lvl_cnt[b, 2] == 0:
            continue
        l = _block_level(lo, hi, cells[b], cam)
        if l >= 0:
            out.append((l, torch.arange(lvl_off[b, l], lvl_off[b, l] + lvl_cnt[b, l], device=DEV)))
    return out


def _exact_lod(case, g):
    levels, lvl_off, lvl_cnt, cells, cams = _city(case, g)
    fine = levels[2][0]
    boxes = [tuple(t.cpu().numpy() for t in _mad_box(fine[:, o:o + c])) if c else (None, None)
             for o, c in zip(lvl_off[:, 2], lvl_cnt[:, 2])]
    if case["half"]:
        for l in (0, 1):
            m, *rest, sh = levels[l]
            levels[l] = (m, *(t.half() for t in rest), sh[:(SH_BANDS[l] + 1) ** 2].half())
    d_rgb = None
    if case["train"]:
        d_rgb = torch.randn((case["views"], 3, case["height"], case["width"]), generator=g, device=DEV)
        grads = [[torch.zeros(t.shape, dtype=torch.float64, device=DEV) for t in lv] for lv in levels]
    rgb, T = [], []
    for v, cam in enumerate(cams):
        pieces = _select(case, levels, lvl_off, lvl_cnt, boxes, cells, cam)
        parts = []
        for l, idx in pieces:
            sel = [t.index_select(t.dim() - 1, idx).double() for t in levels[l]]
            if sel[4].shape[0] < 16:
                sel[4] = torch.cat([sel[4], sel[4].new_zeros((16 - sel[4].shape[0], 3, idx.numel()))])
            parts.append(sel)
        p = [torch.cat([q[k] for q in parts], dim=-1) for k in range(5)]
        a, b, gr = _exact_view(p, cam, 3, 0.0, None if d_rgb is None else d_rgb[v].double())
        rgb.append(a)
        T.append(b)
        at = 0
        for l, idx in pieces if gr is not None else ():
            for k in range(5):
                piece = gr[k][..., at:at + idx.numel()]
                grads[l][k].index_add_(-1, idx, piece[:grads[l][4].shape[0]] if k == 4 else piece)
            at += idx.numel()
    out = {"rgb": torch.stack(rgb), "T": torch.stack(T)}
    if case["train"]:
        out["grads"] = grads
    return out


def _contract(m, box, z):
    """Centres [3, n] normalised to the foreground box and contracted (|c| < 2)."""
    lo = torch.tensor([[box[0]], [box[1]], [z[0]]], dtype=torch.float64, device=DEV)
    hi = torch.tensor([[box[2]], [box[3]], [z[1]]], dtype=torch.float64, device=DEV)
    p = (2.0 * (m.double() - lo)) / (hi - lo) - 1.0
    n = p.abs().amax(dim=0)
    return torch.where(n > 1.0, (2.0 - 1.0 / n) * (p / n), p)


def _block_of(c, grid):
    edges = -2.0 + 4.0 * torch.arange(1, grid, dtype=torch.float64, device=DEV) / grid
    return torch.bucketize(c[1].contiguous(), edges, right=True) * grid + torch.bucketize(c[0].contiguous(), edges,
                                                                                         right=True)


def _exact_setup(case, g):
    arrays, box = _cloud(case, g)
    m, grid = arrays[0], case["grid"]
    block = _block_of(_contract(m, box, (float(m[2].min()), float(m[2].max()))), grid)
    perm = torch.argsort(block, stable=True)
    cnt = torch.bincount(block, minlength=grid * grid)
    ends = torch.cumsum(cnt, 0).cpu().numpy()
    level = [t.index_select(t.dim() - 1, perm) for t in arrays]
    lo, hi, chunks = [], [], []
    for e, c in zip(ends, cnt.cpu().numpy()):
        pts, sc = level[0][:, e - c:e], level[1][:, e - c:e]
        a, b = _mad_box(pts) if c else (torch.full((3,), math.inf, device=DEV, dtype=torch.float64),
                                        torch.full((3,), -math.inf, device=DEV, dtype=torch.float64))
        lo.append(a)
        hi.append(b)
        for q, s in zip(pts.split(2048, dim=1), sc.split(2048, dim=1)) if c else ():
            chunks.append(torch.cat([q.amin(dim=1), q.amax(dim=1), s.abs().max()[None]]))
    chunks += [torch.zeros(7, device=DEV)] * (grid * grid + (case["n"] + 2047) // 2048 - len(chunks))
    return {"perm": None, "off": None, "cells": None, "level": [t.double() for t in level], "lo": torch.stack(lo),
            "hi": torch.stack(hi), "chunk_off": None, "chunks": torch.stack(chunks).double(), "chunk_run": None}


def _ssim(x, y):
    """Mean SSIM of two images [3, H, W] (11 x 11 Gaussian window, sd 1.5, zero padding)."""
    w = torch.exp(-torch.arange(-5, 6, dtype=torch.float64, device=DEV) ** 2 / 4.5)
    w = (w / w.sum())

    def blur(t):
        p = torch.nn.functional.pad(t, (5, 5, 5, 5))
        p = sum(w[k] * p[:, :, k:k + t.shape[2]] for k in range(11))
        return sum(w[k] * p[:, k:k + t.shape[1]] for k in range(11))

    mx, my = blur(x), blur(y)
    sxx, syy, sxy = blur(x * x) - mx * mx, blur(y * y) - my * my, blur(x * y) - mx * my
    return (((2 * mx * my + 1e-4) * (2 * sxy + 9e-4)) / ((mx * mx + my * my + 1e-4) * (sxx + syy + 9e-4))).mean()


def _exact_assign(case, g):
    arrays, box, cams = _assign_inputs(case, g)
    grid, z = case["grid"], arrays[0][2]
    block = _block_of(_contract(arrays[0], box, (float(z.min()), float(z.max()))), grid)
    order = torch.argsort(block, stable=True)
    block = block[order]
    p = [t.index_select(t.dim() - 1, order).double() for t in arrays]
    B = grid * grid
    out = np.ones((len(cams), B))
    with torch.no_grad():
        for k, cam in enumerate(cams):
            flat, rect, depth, which = _project(p, cam, 3)
            of = block[which]
            full = _composite(flat, rect, depth, cam.width, cam.height, 0.0)[0]
            for b in torch.unique(of).tolist():
                keep = of != b
                img = _composite(flat[:, keep], rect[:, keep], depth[keep], cam.width, cam.height, 0.0)[0]
                out[k, b] = float(_ssim(full, img))
    return {"ssim": out, "b": None, "b1": None, "b2": None}


def exact(case, seed):
    g = _gen(seed)
    if case["kind"] == "setup":
        return _exact_setup(case, g)
    if case["kind"] == "assign":
        return _exact_assign(case, g)
    if case["kind"] == "lod":
        return _exact_lod(case, g)
    params, cams = _single_set(case, g)
    p = [t.double() for t in params]
    d_rgb = None
    if case["train"]:
        d_rgb = torch.randn((case["views"], 3, case["height"], case["width"]), generator=g, device=DEV)
    rgb, grads = [], None
    for v, cam in enumerate(cams):
        a, _, gr = _exact_view(p, cam, case["sh_degree"], case["bg"], None if d_rgb is None else d_rgb[v].double())
        rgb.append(a)
        if gr is not None:
            grads = list(gr) if grads is None else [x + y for x, y in zip(grads, gr)]
    out = {"rgb": torch.stack(rgb)}
    if case["train"]:
        out["grads"] = grads
    return out
