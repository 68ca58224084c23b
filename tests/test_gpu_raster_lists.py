"""The raster kernels at the list lengths where their walks change shape: a block's
candidates fill panels of eight, ballots of 64 and staged batches of 128 or more, each
just short, exact and just over, at every tile edge, with and without alphas that reach
the cap.  Image and gradient against the FP64 oracle, with the bars of the parity
tests."""
import numpy as np
import pytest

import scenegen
import oracle
from oracle import composite
from tests import gpu_util as gu

pytestmark = pytest.mark.gpu


def _stack(n, opaque):
    """n Gaussians several pixels across in front of one 24x20 view, so thin that a
    pixel blends nearly all of them; opaque: every ninth one nearly opaque and small."""
    sc = scenegen.small_scene(900 + n, n, 1, [(24, 20)], log_scale_mean=-1.2, half_extent=0.4, bg=(0.3, 0.2, 0.1))
    rng = np.random.default_rng(n)
    sc.params[10, :n] = rng.uniform(-4.4, -3.4, n)
    if opaque:
        sc.params[10, 4:n:9] = rng.uniform(5.0, 9.0, len(range(4, n, 9)))
        sc.params[3:6, 4:n:9] = rng.uniform(-3.4, -2.6, (3, len(range(4, n, 9))))
    return sc


@pytest.mark.parametrize("opaque", [False, True])
@pytest.mark.parametrize("tile", [8, 16, 32])
@pytest.mark.parametrize("n", [1, 4, 7, 8, 9, 63, 64, 65, 72, 127, 128, 129, 260])
def test_list_lengths(n, tile, opaque):
    sc = _stack(n, opaque)
    projs = oracle.project_views(sc.params, sc.n, sc.sh_degree, sc.cams)
    r = composite.render_view(projs[0])
    amb = gu.ambiguous(r)
    up = gu.masked_upstream(scenegen.upstream_grads(n, sc.cams, scale=1e-2), [amb])
    g = gu.run_gpu(sc, upstream=up, tile=tile)
    assert np.abs(g["color"][0] - r["color"]).max(axis=0)[~amb].max() <= 1e-4
    count = gu.split_pixels(sc, g["n_contrib"])[0]
    assert np.array_equal(count[~amb].astype(np.int64), r["n_contrib"][~amb])
    ref = oracle.param_grads(sc.params, sc.n, sc.sh_degree, sc.cams, up)
    for grp, (rel, elem) in gu.grad_errors(g["grad"], ref, np.ones(n, bool), gu.param_groups(1)).items():
        assert rel <= 1e-3 and elem <= 1.0, (grp, rel, elem)
