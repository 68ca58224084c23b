"""The fp32 cutoff test of the binning against the FP64 one (exact mode decides every
candidate tile in FP64): the same pairs in the same order, on splats thin and round,
inside, beside and far larger than the image, opacities around the 1/255 cutoff, images
whose last tiles are one pixel wide, and centres on pixel centres."""
import numpy as np
import pytest

import scenegen
from tests import gpu_util as gu

pytestmark = pytest.mark.gpu


def _scene(seed, n, w, h, grid=False):
    rng = np.random.default_rng(seed)
    sc = scenegen.small_scene(seed, n, 0, [(w, h)], log_scale_mean=-2.6)
    P = sc.params
    P[0:2, :n] = rng.uniform(-1.6, 1.6, (2, n))
    P[3:6, :n] = rng.uniform(-6.5, 0.7, (3, n))          # axes from a fraction of a pixel to the whole image
    P[10, :n] = rng.uniform(-5.55, 4.0, n)               # opacity from just below 1/255
    P[10, : n // 8] = np.log(1 / 254.0) + rng.uniform(-1e-5, 1e-5, n // 8)
    if grid:                                             # screen positions on pixel centres, head on
        c = sc.cams[0]
        c["R"], c["t"] = np.eye(3, dtype=np.float32), np.array([0, 0, 4], np.float32)
        c["fx"] = c["fy"] = np.float32(64.0)
        c["cx"], c["cy"] = np.float32(w / 2), np.float32(h / 2)
        P[2, :n] = 0.0
        P[0, :n] = (rng.integers(-3, w + 3, n) + 0.5 - w / 2) / 16.0
        P[1, :n] = (rng.integers(-3, h + 3, n) + 0.5 - h / 2) / 16.0
        P[3:6, : n // 2] = -3.5
        P[6:10, : n // 2] = np.array([[1.0], [0.0], [0.0], [0.0]])
    return sc


@pytest.mark.parametrize("grid", [False, True])
@pytest.mark.parametrize("tile,w,h", [(16, 97, 65), (8, 97, 65), (32, 97, 65), (16, 16, 16), (8, 1, 9), (16, 640, 17),
                                      (8, 801, 601)])
def test_fp32_test_decides_as_fp64(tile, w, h, grid):
    sc = _scene(tile + w, 3000, w, h, grid)
    a, b = (gu.run_gpu(sc, cull=c, tile=tile) for c in ("ellipse", "exact"))
    assert a["K"] == b["K"] and a["K"] > 0
    for k in ("keys", "values", "pair_view", "ranges"):
        assert np.array_equal(a[k], b[k]), k
