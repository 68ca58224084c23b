"""A non-finite value stays with the pixels and splats that it is blended with.

Of an upstream gradient at one pixel only the splats which that pixel blended get a
non-finite centre, conic or opacity gradient, and only splats that blend into some pixel
of its 8x8 block a non-finite colour gradient; a splat of infinite colour that no pixel of
a block takes (between the pixel centres, of barely more than the cutoff opacity) leaves
the block's image, and every other splat's gradient, as they are.  Everything else is the
same bits as without the value (in the fixed summation order)."""
import numpy as np
import pytest

import scenegen
from tests import gpu_util as gu

pytestmark = pytest.mark.gpu

W, H = 56, 40


def _scene(n=300, opaque=False):
    """Head on at 16 pixels a unit: splat g's centre is where its parameters say."""
    sc = scenegen.small_scene(77, n, 0, [(W, H)], bg=(0.2, 0.4, 0.6))
    rng = np.random.default_rng(5)
    c = sc.cams[0]
    c["R"], c["t"] = np.eye(3, dtype=np.float32), np.array([0, 0, 4], np.float32)
    c["fx"] = c["fy"] = np.float32(64.0)
    P = sc.params
    P[0], P[1] = rng.uniform(-W / 32, W / 32, n), rng.uniform(-H / 32, H / 32, n)
    P[2] = rng.uniform(-0.5, 0.5, n)
    P[3:6] = rng.uniform(-4.0, -1.8, (3, n))
    P[10] = rng.uniform(-4.0, 1.0, n)
    if opaque:
        P[10, ::7] = 6.0
    return sc


def _exponents(g):
    """[n, H, W] exponents and whether a pixel's centre is clearly outside a splat's cutoff."""
    u, w, a, b, c, tau = (g[k][0].astype(np.float64)[:, None, None] for k in ("u", "w", "a", "b", "c", "tau"))
    dx, dy = u - (np.arange(W)[None, None, :] + 0.5), w - (np.arange(H)[None, :, None] + 0.5)
    p = -0.5 * (a * dx * dx + c * dy * dy) - b * dx * dy
    return p < tau - 1e-3


def _block_any(m, x, y):
    return m[:, y // 8 * 8: y // 8 * 8 + 8, x // 8 * 8: x // 8 * 8 + 8].reshape(m.shape[0], -1)


@pytest.mark.parametrize("opaque", [False, True])
@pytest.mark.parametrize("value", [np.inf, np.nan, 3e38])
@pytest.mark.parametrize("tile", [8, 16, 32])
def test_upstream_gradient_of_one_pixel(tile, value, opaque):
    sc = _scene(opaque=opaque)
    up = scenegen.upstream_grads(3, sc.cams, 1e-2)
    clean = gu.run_gpu(sc, upstream=up, tile=tile, bwd="ordered")
    x, y = 21, 19
    up[0][:, y, x] = value
    dirty = gu.run_gpu(sc, upstream=up, tile=tile, bwd="ordered")
    off = _exponents(clean)
    not_here = off[:, y, x]                                    # not blended at the pixel
    not_block = _block_any(off, x, y).all(1)                   # nor anywhere in its block
    a, b = (r["grad2d"].reshape(sc.n, 9).view(np.uint32) for r in (clean, dirty))
    assert not_here.sum() > 100 and (~not_here).sum() > 5 and (not_here & ~not_block).sum() > 10
    assert np.array_equal(a[not_here, :6], b[not_here, :6])
    assert np.array_equal(a[not_block], b[not_block])
    assert not np.isfinite(dirty["grad2d"].reshape(sc.n, 9)[~not_here]).all()


@pytest.mark.parametrize("opaque", [False, True])
@pytest.mark.parametrize("value", [np.inf, np.nan])
@pytest.mark.parametrize("tile", [8, 16, 32])
def test_colour_of_a_splat_that_no_pixel_takes(tile, value, opaque):
    sc = _scene(opaque=opaque)
    rng = np.random.default_rng(9)
    k = 40
    P = sc.params
    P[0, :k] = (rng.integers(1, W, k) - W / 2) / 16            # between pixel centres
    P[1, :k] = (rng.integers(1, H, k) - H / 2) / 16
    P[2, :k] = rng.choice([-1.0, 1.0], k) * 1e-3
    P[0, :k] *= (4 + P[2, :k]) / 4
    P[1, :k] *= (4 + P[2, :k]) / 4
    P[3:6, :k] = -9.0                                          # the cutoff region: 0.1 pixels across
    o = 1.005 / 255
    P[10, :k] = np.log(o / (1 - o))
    up = scenegen.upstream_grads(3, sc.cams, 1e-2)
    clean = gu.run_gpu(sc, upstream=up, tile=tile, bwd="ordered")
    P[11:14, :k] = value
    dirty = gu.run_gpu(sc, upstream=up, tile=tile, bwd="ordered")
    off = _exponents(clean)
    assert off[:k].all() and not off[k:].all()
    assert dirty["K"] == clean["K"] and (clean["values"] < k).sum() >= k // 2
    assert np.array_equal(clean["color"][0].view(np.uint32), dirty["color"][0].view(np.uint32))
    for key in ("n_contrib", "last", "evals"):
        assert np.array_equal(clean[key], dirty[key]), key
    assert np.array_equal(clean["grad2d"].view(np.uint32), dirty["grad2d"].view(np.uint32))
