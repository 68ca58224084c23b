"""A non-finite value stays with the pixels and splats that it is blended with.

Of an upstream gradient at one pixel only the splats which that pixel blended get a
non-finite centre, conic or opacity gradient, and only splats that blend into some pixel
of its 8x8 block a non-finite colour gradient.  Everything else is the same bits as
without the value (in the fixed summation order)."""
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
@pytest.mark.parametrize("value", [np.inf, -np.inf, np.nan, 3e38])
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
