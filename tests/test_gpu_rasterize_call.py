"""What GaussianRasterize.apply takes and keeps."""
import numpy as np
import pytest
import torch

from paper_2404_01133_amd import gs, render, synth

pytestmark = pytest.mark.gpu


def _case(n=2_000, V=3, width=90, height=50):
    g = synth.box_gaussians(n, seed=3, extent=((-20, 20), (-20, 20), (0, 8)))
    cams = synth.orbit_views((0.0, 0.0), n_views=V, radius=30.0, height=25.0, width=width, h_px=height)
    return [torch.from_numpy(np.ascontiguousarray(a)).cuda() for a in g.astuple()], cams


@pytest.mark.parametrize("views", [1, 2])
def test_cameras_beyond_n_views_are_not_read(views):
    """The first n_views cameras of a longer buffer, as gs_preprocess takes them."""
    arrays, cams = _case()
    one = gs.cameras_to_device(cams[:views])
    more = gs.cameras_to_device(cams)
    a, b = (render.GaussianRasterize.apply(*arrays, c, views, 90, 50, 3, (0.0, 0.0, 0.0), None) for c in (one, more))
    assert float(a.abs().max()) > 0 and torch.equal(a, b)
    padded = torch.cat([one, torch.full((16,), 0x55, dtype=torch.uint8, device="cuda")])
    assert torch.equal(a, render.GaussianRasterize.apply(*arrays, padded, views, 90, 50, 3, (0.0, 0.0, 0.0), None))


def test_gradients_through_apply_equal_those_of_rasterize():
    """Called with and without the block table: the same twelve or thirteen arguments back."""
    arrays, cams = _case()
    d = torch.from_numpy(np.random.default_rng(1).normal(size=(3, 3, 50, 90)).astype(np.float32)).cuda()
    got = []
    for call in (lambda p: render.rasterize(*p, cams),
                 lambda p: render.GaussianRasterize.apply(*p, gs.cameras_to_device(cams), 3, 90, 50, 3,
                                                          (0.0, 0.0, 0.0), None)):
        p = [a.clone().requires_grad_() for a in arrays]
        call(p).backward(d)
        got.append([t.grad.double() for t in p])
    for a, b in zip(*got):  # sums of the same FP32 terms in another order
        assert float(b.norm()) > 0 and float((a - b).norm()) <= 1e-5 * float(b.norm())


@pytest.mark.parametrize("n", [500, 100_000])
def test_memory_held_for_the_backward(n):
    """Between forward and backward, autograd holds no more of a frame of its own than a frame of 4 pairs a
    record takes, and up to 8 MB of room for pairs that is not worth a copy; the gradients are those through
    a kept frame."""
    g = synth.cube_gaussians(n, 3)
    g.scales = (g.scales * 0.05).astype(np.float32)
    cams = [synth.axis_camera(200, 120)] * 2
    arrays = [torch.from_numpy(np.ascontiguousarray(a)).cuda() for a in g.astuple()]
    d = torch.from_numpy(np.random.default_rng(1).normal(size=(2, 3, 120, 200)).astype(np.float32)).cuda()

    def allocated():
        torch.cuda.synchronize()
        return torch.cuda.memory_allocated()
    start = allocated()
    frame = render.Frame(1, 2, 200, 120, 2 * n, max(4096, 8 * n))
    of_frame = allocated() - start
    p = [a.clone().requires_grad_() for a in arrays]
    render.rasterize(*p, cams, frame=frame).backward(d)
    want = [t.grad.double() for t in p]
    p = [a.clone().requires_grad_() for a in arrays]
    start = allocated()
    img = render.rasterize(*p, cams)
    held = allocated() - start
    print("case:", n, "held", held, "frame", of_frame, "pairs", frame.pairs, flush=True)
    assert frame.pairs <= 8 * n and held <= of_frame + img.numel() * 4 + 4096 + (8 << 20)  # (cameras and table)
    img.backward(d)
    for a, t in zip(want, p):  # sums of the same FP32 terms in another order
        assert float(a.norm()) > 0 and float((a - t.grad.double()).norm()) <= 1e-5 * float(a.norm())
