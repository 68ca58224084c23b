"""The SSIM loss at the shapes where its tiles end: widths around the 44 columns of a
tile and the window's reach, heights around the window and a tile's rows, several views
in one launch, strips enough that the channels of a tile share a sum, values
outside [0, 1], and a gradient written over an image.  Against the oracle at the loss's
parity bar: values to 1e-6 relative, dL/dimage to 1e-4 of its largest value."""
import numpy as np
import pytest
import torch

import oracle
import paper_2503_13086_amd as gs
import scenegen
from paper_2503_13086_amd.pipeline import Rasterizer, params_to_device

pytestmark = pytest.mark.gpu


def _images(rng, sizes, lo=0.0, hi=1.0):
    xn = [rng.uniform(lo, hi, (3, h, w)).astype(np.float32) for w, h in sizes]
    yn = [(a + rng.normal(0, 0.1, a.shape)).astype(np.float32) for a in xn]
    return xn, yn


def _views(rz, sizes):
    sc = scenegen.small_scene(3, 4, 0, [(16, 16)])
    cams = [scenegen.pinhole(np.eye(3), np.array([0.0, 0.0, 3.0]), w, h, 0.9, (0.0, 0.0, 0.0)) for w, h in sizes]
    rz.preprocess(params_to_device(sc.params), sc.n, 0, cams)


def _check(sizes, xn, yn, loss, dl, w_l1, w_dssim):
    off = 0
    for v, (w, h) in enumerate(sizes):
        val, grad = oracle.image_loss_and_grad(xn[v], yn[v], w_l1, w_dssim)
        assert abs(loss[v] - val) <= 1e-6 * abs(val) + 1e-9, (v, loss[v], val)
        got = dl[off: off + 3 * w * h].reshape(3, h, w)
        assert np.abs(got - grad).max() <= 1e-4 * np.abs(grad).max(), v
        off += 3 * w * h


SHAPES = [[(1, 1)], [(5, 3)], [(11, 11)], [(43, 12)], [(44, 12)], [(45, 13)], [(88, 24)], [(89, 33)], [(64, 34)],
          [(133, 35)], [(1, 200)], [(700, 1)], [(97, 154)], [(44, 45), (1, 7), (131, 67), (40, 12)],
          [(16384, 1)] * 60]


@pytest.mark.parametrize("sizes", SHAPES, ids=lambda s: "%d_of_%dx%d" % (len(s), *s[0]))
def test_shapes(sizes):
    rng = np.random.default_rng(len(sizes) + sizes[0][0])
    rz = Rasterizer(0)
    try:
        _views(rz, sizes)
        xn, yn = _images(rng, sizes, -0.5, 1.5)
        x, y = rz.pack_images(xn), rz.pack_images(yn)
        for call in (gs.gs_loss, gs.gs_loss_noalloc):
            lo = torch.zeros(len(sizes), dtype=torch.float64, device=rz.device)
            dl = rz.new_image(fill=7.0)
            call(rz.ctx, x, y, 0.8, 0.2, lo, dl)
            torch.cuda.synchronize()
            _check(sizes, xn, yn, lo.cpu().numpy(), dl.cpu().numpy(), 0.8, 0.2)
    finally:
        rz.close()


@pytest.mark.parametrize("over", ["color", "target"])
def test_gradient_over_an_image(over):
    sizes = [(150, 101), (77, 45)]
    rng = np.random.default_rng(5)
    rz = Rasterizer(0)
    try:
        _views(rz, sizes)
        xn, yn = _images(rng, sizes)
        x, y = rz.pack_images(xn), rz.pack_images(yn)
        lo = torch.zeros(len(sizes), dtype=torch.float64, device=rz.device)
        dl = x if over == "color" else y
        gs.gs_loss(rz.ctx, x, y, 0.8, 0.2, lo, dl)
        torch.cuda.synchronize()
        _check(sizes, xn, yn, lo.cpu().numpy(), dl.cpu().numpy(), 0.8, 0.2)
    finally:
        rz.close()


def test_nan_and_infinite_pixels_stay_where_the_windows_reach():
    w, h = 150, 90
    rng = np.random.default_rng(6)
    rz = Rasterizer(0)
    try:
        _views(rz, [(w, h)])
        xn, yn = _images(rng, [(w, h)])
        clean = oracle.image_loss_and_grad(xn[0], yn[0], 0.8, 0.2)[1]
        xn[0][1, 40, 60] = np.nan
        xn[0][2, 70, 100] = np.inf
        dl = rz.new_image(fill=7.0)
        gs.gs_loss(rz.ctx, rz.pack_images(xn), rz.pack_images(yn), 0.8, 0.2, None, dl)
        torch.cuda.synchronize()
        got = dl.cpu().numpy().reshape(3, h, w)
        reach = np.zeros((3, h, w), bool)
        reach[1, 30:51, 50:71] = True
        reach[2, 60:81, 90:111] = True
        assert np.abs(got - clean)[~reach].max() <= 1e-4 * np.abs(clean).max()
        assert not np.isfinite(got[1, 40, 60]) and not np.isfinite(got[2, 70, 100])
    finally:
        rz.close()
