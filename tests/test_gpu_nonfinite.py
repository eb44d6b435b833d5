"""Colours that are not finite reach the gradients of the pixels that show them and no others; an infinite
opacity is a clamped one.

Two faint splats of under a pixel, one in the upper two rows of a 4x4 quadrant, one in the lower
two: neither reaches a pixel of the other, while the adjoint walks both for all sixteen pixels.  The
front one's colour is infinite or NaN; image and gradients of the other one have to be those it has alone."""
import numpy as np
import pytest
import torch

from paper_2404_01133_amd import gs, render, synth

pytestmark = pytest.mark.gpu

W = H = 32


def _splats(cam, px, depth):
    """Round splats of 0.01 px centred at pixel coordinates px (K, 2), opacity 4/255."""
    px, z = np.asarray(px, float), np.asarray(depth, float)
    n = len(z)
    means = np.stack([(px[:, 0] - cam.cx) / cam.fx * z, (px[:, 1] - cam.cy) / cam.fy * z, z - cam.t[2]])
    quats = np.zeros((4, n))
    quats[0] = 1.0
    sh = np.random.default_rng(3).normal(size=(16, 3, n)) * 0.2
    sh[0] += 1.0
    return [np.ascontiguousarray(a, np.float32) for a in
            (means, np.full((3, n), 0.01 / cam.fx), quats, np.full(n, 4.0 / 255.0), sh)]


def _render(arrays, cam, tuning, d):
    p = [torch.from_numpy(a).cuda().requires_grad_() for a in arrays]
    frame = render.Frame(1, 1, W, H, 2, 256, tuning)
    img = render.rasterize(*p, [cam], frame=frame)
    img.backward(d)
    return img.detach().cpu().numpy()[0], [t.grad.cpu().numpy() for t in p]


@pytest.mark.parametrize("flags", [0, gs.GS_TUNE_DETERMINISTIC])
@pytest.mark.parametrize("tile,batch", [((16, 16), 256), ((8, 8), 64), ((32, 16), 128)])
@pytest.mark.parametrize("colour", [np.inf, np.nan])
def test_other_splats_of_the_quadrant_are_untouched(colour, tile, batch, flags):
    cam = synth.axis_camera(W, H)
    tuning = gs.tuning_struct(tile[0], tile[1], batch, flags)
    both = _splats(cam, [(10.0, 9.0), (10.0, 11.0)], [3.0, 4.0])  # rows 8 and 9, rows 10 and 11
    both[4][0, 1, 0] = colour
    alone = [np.ascontiguousarray(a[..., 1:]) for a in both]
    d = torch.from_numpy(np.random.default_rng(5).normal(size=(1, 3, H, W)).astype(np.float32)).cuda()
    img, got = _render(both, cam, tuning, d)
    want_img, want = _render(alone, cam, tuning, d)
    assert np.abs(want_img[:, 10:12]).max() > 0 and not np.isfinite(img[1, 8:10]).all()
    np.testing.assert_array_equal(img[:, 10:], want_img[:, 10:])
    assert all(np.isfinite(b).all() for b in want)
    assert all(np.abs(want[k]).max() > 0 for k in (0, 1, 3, 4))  # (a round splat's rotation has no gradient)
    for a, b in zip(got, want):  # the same pixels, the same operations: equal bits
        np.testing.assert_array_equal(a[..., 1], b[..., 0])


@pytest.mark.parametrize("flags", [0, gs.GS_TUNE_DETERMINISTIC])
@pytest.mark.parametrize("opacity", [np.inf, 3.0e38])
def test_opacity_beyond_the_clamp(opacity, flags):
    """An alpha that is clamped at every pixel of the splat depends on neither opacity nor shape: those gradients
    are exactly 0, everything else is as with any other opacity that large."""
    cam = synth.axis_camera(W, H)
    tuning = gs.tuning_struct(16, 16, 256, flags)
    d = torch.from_numpy(np.random.default_rng(5).normal(size=(1, 3, H, W)).astype(np.float32)).cuda()
    arrays = _splats(cam, [(10.0, 9.0), (11.0, 10.0)], [3.0, 4.0])
    arrays[1][:] = 0.002  # under a pixel: with 0.3 px^2 of dilation exp2(-Q) >= 1e-10 in the 4x4 pixels of the footprint
    arrays[3][:] = 1.0e30, 0.5
    _, want = _render(arrays, cam, tuning, d)
    arrays[3][0] = opacity
    img, got = _render(arrays, cam, tuning, d)
    assert np.isfinite(img).all()
    for a, b in zip(got, want):
        np.testing.assert_array_equal(a, b)
    for k in (1, 2, 3):
        assert np.all(got[k][..., 0] == 0.0) and np.isfinite(got[k]).all()
    assert np.abs(got[4][..., 0]).max() > 0 and np.abs(got[1][..., 1]).max() > 0


@pytest.mark.parametrize("tile,batch,flags", [((16, 16), 256, 0), ((8, 8), 64, gs.GS_TUNE_WORK_QUEUE),
                                              ((32, 16), 128, 0)])
@pytest.mark.parametrize("colour", [np.inf, np.nan])
def test_image_shows_it_where_it_is_used_only(colour, tile, batch, flags):
    """Neither a pixel of the same group that the splat does not reach nor one that is done before it changes."""
    cam = synth.axis_camera(W, H)
    tuning = gs.tuning_struct(tile[0], tile[1], batch, flags)
    d = torch.zeros((1, 3, H, W), device="cuda")
    faint = _splats(cam, [(10.0, 9.0), (22.0, 21.0)], [3.0, 4.0])
    want, _ = _render(faint, cam, tuning, d)
    faint[4][0, 1, 0] = colour
    got, _ = _render(faint, cam, tuning, d)
    reached = np.zeros((H, W), bool)
    reached[8:10, 9:11] = True
    assert np.all(want[:, reached] > 0) and not np.isfinite(got[1][reached]).any()
    np.testing.assert_array_equal(got[1][~reached], want[1][~reached])
    np.testing.assert_array_equal(got[[0, 2]], want[[0, 2]])
    # 300 splats of every opacity up to the clamp over the left half, one behind them over everything
    rng = np.random.default_rng(9)
    px = np.stack([rng.uniform(0, 16, 300), rng.uniform(0, H, 300)], 1)
    px = np.concatenate([px, [[16.0, 16.0]]])
    many = _splats(cam, px, np.concatenate([rng.uniform(1.0, 3.0, 300), [4.0]]))
    many[1][:, :300] = 2.0 / cam.fx
    many[1][:, 300] = 100.0
    many[3][:300] = rng.uniform(0.3, 1.0, 300)
    many[3][300] = 0.5
    front = [np.ascontiguousarray(a[..., :300]) for a in many]
    want, _ = _render(many, cam, tuning, d)
    many[4][0, :, 300] = colour
    got, _ = _render(many, cam, tuning, d)
    alone, _ = _render(front, cam, tuning, d)
    used = (want != alone).any(0)  # (where the last splat shows)
    assert used.any() and not used.all() and not np.isfinite(got[:, used]).any()
    np.testing.assert_array_equal(got[:, ~used], want[:, ~used])
