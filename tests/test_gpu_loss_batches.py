"""A view's loss value and gradient are the same bits alone and in any batch, and from
gs_loss and gs_loss_noalloc, whatever strips the launch is cut into."""
import numpy as np
import pytest
import torch

import paper_2503_13086_amd as gs
import scenegen
from paper_2503_13086_amd.pipeline import Rasterizer, params_to_device

pytestmark = pytest.mark.gpu


def _views(rz, sizes):
    sc = scenegen.small_scene(3, 4, 0, [(16, 16)])
    cams = [scenegen.pinhole(np.eye(3), np.array([0.0, 0.0, 3.0]), w, h, 0.9, (0.0, 0.0, 0.0)) for w, h in sizes]
    rz.preprocess(params_to_device(sc.params), sc.n, 0, cams)


def _images(px, seed):
    g = torch.Generator(device="cuda").manual_seed(seed)
    x = torch.rand(3 * px, generator=g, device="cuda")
    return x, (x + 0.1 * torch.randn(3 * px, generator=g, device="cuda")).clamp(0.0, 1.0)


def _loss(rz, sizes, x, y, w_l1, w_dssim, call=gs.gs_loss):
    _views(rz, sizes)
    lo = torch.full((len(sizes),), -1.0, dtype=torch.float64, device="cuda")
    dl = torch.full_like(x, 7.0)
    call(rz.ctx, x, y, w_l1, w_dssim, lo, dl)
    torch.cuda.synchronize()
    return lo.cpu().numpy(), dl


# batches from one strip height to the tallest: one to nine large views, ragged ones,
# small ones by the dozen, and one that has more tiles than the chip holds several times
BATCHES = [[(1296, 864)] * 2, [(1296, 864)] * 6, [(1600, 1067), (1296, 864), (979, 546)] * 3,
           [(333, 217), (250, 131), (197, 301)], [(700, 500), (45, 700), (1, 9), (1600, 1067)] * 5,
           [(96, 64)] * 64, [(4001, 3001), (979, 546)]]


@pytest.mark.parametrize("sizes", BATCHES, ids=lambda s: "%d_of_%dx%d" % (len(s), *s[0]))
def test_alone_equals_batch(sizes):
    px = [w * h for w, h in sizes]
    x, y = _images(sum(px), len(sizes))
    rz = Rasterizer(0)
    try:
        lo, dl = _loss(rz, sizes, x, y, 0.47, 0.12)
        ln, dn = _loss(rz, sizes, x, y, 0.47, 0.12, gs.gs_loss_noalloc)
        assert np.array_equal(lo, ln) and torch.equal(dl, dn)
        off = 0
        for v, p in enumerate(px):
            one, d1 = _loss(rz, sizes[v: v + 1], x[3 * off: 3 * (off + p)], y[3 * off: 3 * (off + p)], 0.47, 0.12)
            assert one[0] == lo[v], (v, sizes[v], one[0], lo[v])
            assert torch.equal(d1, dl[3 * off: 3 * (off + p)]), v
            off += p
    finally:
        rz.close()
