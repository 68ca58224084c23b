"""The binning's sorts at the sizes where their shape changes: entries around one
4096-item block, around the 128 blocks up to which a pass adds its table's rows and the
1024 up to which it adds their chunk sums, the 256 whose sums the scan's last workgroup
adds up, tile ids of one, two and three digits, and depths whose bit patterns span from
nothing to the whole range of positive floats.  Every listed pair is enumerated in numpy
from the projection's tile rects and ordered by (tile, depth, index); keys, values, views
and ranges must be equal bit for bit."""
import numpy as np
import pytest
import torch

import paper_2503_13086_amd as gs
import scenegen
from paper_2503_13086_amd.pipeline import Rasterizer, params_to_device

pytestmark = pytest.mark.gpu


def _field(n, seed, depth=None):
    """n small Gaussians in front of a camera at the origin; depth: their camera depths
    (default: uniform in 2..4, many equal)."""
    rng = np.random.default_rng(seed)
    P = scenegen.make_field(rng, n, 0, log_scale_mean=-6.0, log_scale_std=0.3)
    z = np.round(rng.uniform(2.0, 4.0, n), 3) if depth is None else depth
    P[0:2, :n] = rng.uniform(-0.6, 0.6, (2, n)) * z
    P[2, :n] = z
    P[3:6, :n] += np.log(np.maximum(z, 1e-3))        # the same size on screen at any depth
    return P


def _check(P, n, cams, tile):
    rz = Rasterizer(0)
    try:
        gs.gs_set_cull(rz.ctx, gs.GS_CULL_RECT)
        rz.set_views(cams, tile)
        rz.preprocess(params_to_device(P), n, 0)
        K = rz.bin_sort()
        V = len(cams)
        rect = rz.buffer(gs.GS_BUF_TILE_RECT).cpu().numpy().view(np.uint16).reshape(V, n, 4).astype(np.int64)
        touched = rz.buffer(gs.GS_BUF_TOUCHED).cpu().numpy().reshape(V, n)
        depth = rz.buffer(gs.GS_BUF_DEPTH).cpu().numpy().view(np.uint32).reshape(V, n)
        tiles, deps, idx, views = [], [], [], []
        for v, c in enumerate(cams):
            tx = -(-c["width"] // tile)
            x0, x1, y0, y1 = rect[v].T
            for dy in range(int((y1 - y0).max()) + 1):
                for dx in range(int((x1 - x0).max()) + 1):
                    g = np.nonzero((touched[v] > 0) & (x0 + dx <= x1) & (y0 + dy <= y1))[0]
                    tiles.append(rz.tile_off[v] + (y0[g] + dy) * tx + x0[g] + dx)
                    deps.append(depth[v, g])
                    idx.append(g)
                    views.append(np.full(len(g), v))
        tiles, deps, idx, views = (np.concatenate(x) for x in (tiles, deps, idx, views))
        order = np.lexsort((idx, deps, tiles))
        keys = (tiles.astype(np.uint64) << np.uint64(32)) | deps.astype(np.uint64)
        assert K == len(order)
        got = {k: rz.buffer(b).cpu().numpy() for k, b in (("keys", gs.GS_BUF_KEYS), ("values", gs.GS_BUF_VALUES),
                                                          ("views", gs.GS_BUF_PAIR_VIEW), ("ranges", gs.GS_BUF_RANGES))}
        assert np.array_equal(got["keys"].view(np.uint64), keys[order])
        assert np.array_equal(got["values"].astype(np.int64), idx[order])
        assert np.array_equal(got["views"].astype(np.int64), views[order])
        count = np.bincount(tiles, minlength=rz.tile_off[-1])
        end = np.cumsum(count)
        r = got["ranges"].reshape(-1, 2).astype(np.int64)
        assert np.array_equal(r[:, 1] - r[:, 0], count)
        assert np.array_equal(r[count > 0, 1], end[count > 0])
        torch.cuda.synchronize()
    finally:
        rz.close()


def _cam(w, h, f=1.0):
    return scenegen.camera(np.eye(3), np.zeros(3), f * w, f * w, w / 2, h / 2, w, h)


@pytest.mark.parametrize("n", [1, 63, 4095, 4096, 4097, 3 * 4096 + 5, 128 * 4096, 128 * 4096 + 1, 256 * 4096,
                               256 * 4096 + 1])
def test_entry_counts(n):
    _check(_field(n, n), n, [_cam(128, 96)], 16)


@pytest.mark.parametrize("n", [512 * 4096, 512 * 4096 + 1])
def test_entry_counts_two_views(n):
    _check(_field(n, n), n, [_cam(128, 96), _cam(96, 96)], 16)


@pytest.mark.parametrize("size,tile", [((16, 16), 16), ((40, 24), 8), ((300, 200), 8), ((1600, 900), 8),
                                       ((3000, 2900), 8), ((4090, 4080), 8)])
def test_tile_id_widths(size, tile):
    """1 and 15 tiles (one digit), 950 and 22 600 (two, packed into one word), 136 000 and
    261 000 (three); and twice as many in two views."""
    n = 20_000
    _check(_field(n, 5), n, [_cam(*size)], tile)
    _check(_field(n, 6), n, [_cam(*size), _cam(size[0] - 3, size[1])], tile)


@pytest.mark.parametrize("lo,hi", [(1.0, 1.0), (1.0, 1.0000002), (3.0, 3.1), (0.21, 5e4), (0.21, 1e9), (1e3, 1e20),
                                   (0.21, 1e36)])
def test_depth_spans(lo, hi):
    n = 9000
    rng = np.random.default_rng(11)
    z = np.exp(rng.uniform(np.log(lo), np.log(hi), n)).astype(np.float32)
    z[:3], z[3:6] = lo, hi
    z[6] = -1.0                                   # one behind the camera
    P = _field(n, 12, z)
    _check(P, n, [_cam(64, 64)], 16)


def test_nothing_visible():
    n = 5000
    P = _field(n, 13, np.full(n, -2.0))
    rz = Rasterizer(0)
    try:
        rz.preprocess(params_to_device(P), n, 0, [_cam(64, 64)])
        assert rz.bin_sort() == 0
        assert not rz.buffer(gs.GS_BUF_RANGES).cpu().numpy().any()
    finally:
        rz.close()
