"""The projection and its adjoint where a wave holds Gaussians of several levels and
views, and on both sides of the number of views whose constants are kept in LDS (32)."""

import numpy as np
import pytest
import torch

from gpu_util import scaled_city
from paper_2404_01133_amd import gs, render, synth

pytestmark = pytest.mark.gpu


def _frame_and_grads(scene, cams_dev, V, flags, d):
    frame = render.Frame(64, V, 64, 48, V * scene.max_records_per_view(), 1 << 19,
                         gs.tuning_struct(16, 16, 256, flags))
    render.render_frame(scene, frame, cams_dev, thresholds=(300.0, 450.0))
    grads = [lv.zeros_like() for lv in scene.levels]
    render.backward_frame(scene, frame, cams_dev, d, grads)
    return frame, [[t.double().cpu().numpy() for t in (g.means, g.scales, g.quats, g.opac, g.sh)] for g in grads]


@pytest.mark.parametrize("V", [2, 32, 33])
def test_gaussian_major_equals_view_major_with_mixed_levels(V):
    """All views have one camera, so they select the same blocks at the same, different levels; about
    30 Gaussians a block, so that a wave spans blocks, levels and (view-major) views.  Images are
    equal; gradients are sums of the same V terms in another order."""
    bs = scaled_city(2_000, seed=5)
    scene = render.DeviceScene.from_block_scene(bs)
    scene.compute_bounds(4.0)
    cams_dev = gs.cameras_to_device([synth.look_camera((0.0, 0.0, 250.0), 0.3, -0.7, 64, 48)] * V)
    d = torch.from_numpy(np.random.default_rng(V).normal(size=(1, 3, 48, 64)).astype(np.float32)).cuda()
    d = d.expand(V, 3, 48, 64).contiguous()
    shared, got = _frame_and_grads(scene, cams_dev, V, gs.GS_TUNE_SHARED_SELECTION, d)
    plain, want = _frame_and_grads(scene, cams_dev, V, 0, d)
    levels = shared.level.view(V, -1)[0]
    assert len(set(levels[levels >= 0].tolist())) > 1
    assert torch.equal(shared.rgb, plain.rgb) and float(shared.rgb.abs().max()) > 0
    # sums of the same FP32 terms in another order, as wherever two runs are compared: 1e-5 relative
    for a, b in zip(got, want):
        for x, y in zip(a, b):
            assert np.linalg.norm(x - y) <= 1e-5 * np.linalg.norm(y)


@pytest.mark.parametrize("side_stream", [False, True])
def test_rasterize_equals_apply_with_cameras_alone(side_stream):
    """rasterize() sends cameras and block table in one copy on the current stream;
    the function also takes cameras without the table.  Same images, kept apart from the frame's."""
    g = synth.box_gaussians(3_000, seed=3, extent=((-20, 20), (-20, 20), (0, 8)))
    cams = synth.orbit_views((0.0, 0.0), n_views=3, radius=30.0, height=25.0, width=90, h_px=50)
    arrays = [torch.from_numpy(np.ascontiguousarray(a)).cuda() for a in g.astuple()]
    cams_dev = gs.cameras_to_device(cams)
    torch.cuda.synchronize()
    stream = torch.cuda.Stream() if side_stream else torch.cuda.current_stream()
    with torch.cuda.stream(stream):
        frame = render.Frame(1, 3, 90, 50, 3 * 3_000, 1 << 12)  # too few pairs: the frame is rendered again
        a = render.rasterize(*arrays, cams, frame=frame)
        b = render.GaussianRasterize.apply(*arrays, cams_dev, 3, 90, 50, 3, (0.0, 0.0, 0.0), None)
    stream.synchronize()
    assert frame.pair_capacity > 1 << 12 and float(a.abs().max()) > 0
    assert torch.equal(a, b) and torch.equal(a, frame.rgb) and a.data_ptr() != frame.rgb.data_ptr()
