"""Splats below the cutoff opacity 1/255 (and of no opacity at all) blend into no pixel,
whichever tiles list them (gs_set_cull).  As needles of thousands of pixels whose centre
lies as far off the image: their fp32 conic is indefinite by rounding there, so the
exponent that a pixel forms can have either sign and any small size."""
import numpy as np
import pytest

import scenegen
from tests import gpu_util as gu

pytestmark = pytest.mark.gpu


def _needles(n, size, seed=11):
    """Needles at depth 4 (16 pixels a unit) that cross the view, centred off its left side."""
    sc = scenegen.small_scene(seed, n, 0, [(size, size)], bg=(0.25, 0.5, 0.75))
    rng = np.random.default_rng(seed)
    c = sc.cams[0]
    c["R"], c["t"] = np.eye(3, dtype=np.float32), np.array([0, 0, 4], np.float32)
    c["fx"] = c["fy"] = np.float32(64.0)
    th = rng.uniform(0.2, 1.37, n)
    x, y = rng.uniform(0, size, n), rng.uniform(0, size, n)      # a pixel the needle crosses
    u = rng.uniform(-6000, -1500, n)
    P = sc.params
    P[0], P[1], P[2] = (u - size / 2) / 16, (y + (u - x) * np.tan(th) - size / 2) / 16, 0.0
    P[3] = np.log(rng.uniform(1500, 9000, n) / 16)
    P[4:6] = -7.0
    P[6], P[7:9], P[9] = np.cos(th / 2), 0.0, np.sin(th / 2)
    o = rng.uniform(0.0015, 0.0038, n)
    P[10] = np.log(o / (1 - o))
    return sc


@pytest.mark.parametrize("opacity", ["faint", "nan"])
@pytest.mark.parametrize("cull", ["rect", "ellipse"])
@pytest.mark.parametrize("tile", [8, 16, 32])
def test_nothing_blends(tile, cull, opacity):
    sc = _needles(1000, 256)
    if opacity == "nan":
        sc.params[10, ::2] = np.nan
    g = gu.run_gpu(sc, upstream=scenegen.upstream_grads(3, sc.cams, 1e-2), cull=cull, tile=tile)
    assert g["K"] > 30_000 if cull == "rect" else g["K"] == 0
    assert not g["n_contrib"].any() and not g["last"].any() and (g["T_final"] == 1.0).all()
    assert not g["evals"].any() and not g["pairs_eff"].any()
    assert np.array_equal(g["color"][0], np.broadcast_to(sc.cams[0]["bg"][:, None, None], g["color"][0].shape))
    assert not g["grad2d"].any()
