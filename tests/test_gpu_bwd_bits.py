"""In the fixed summation order a backward is the same bits stored, written by the fused
step or applied by it, and the fused step the same as the backward and then the Adam step
(gs_set_backward_order, gs_render_bwd_adam)."""
import numpy as np
import pytest

from tests.test_gpu_bwd_views import _run, _scene

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("views", [1, 2, 3])
@pytest.mark.parametrize("sh", [0, 1, 2, 3])
@pytest.mark.parametrize("n", [257, 3000])
def test_fused_equals_separate(n, sh, views):
    sc = _scene(n, sh, ((61, 45), (40, 52), (33, 70))[:views])
    sep, acc = _run(sc, sc.cams, "separate", n), _run(sc, sc.cams, "accumulate", n)
    f32 = lambda a: a.astype(np.float32)
    assert np.array_equal(f32(acc["grad"]), f32(acc["base"]) + f32(sep["grad"]))
    for mode in ("fused", "fused_grad"):
        f = _run(sc, sc.cams, mode, n)
        if mode == "fused_grad":
            d = f["grad"] != sep["grad"]
            assert not d.any(), (mode, "grad", int(d.sum()), np.nonzero(d.any(1))[0])
        for k in ("P", "m", "v", "step"):
            d = f[k] != sep[k]
            assert not d.any(), (mode, k, int(d.sum()), np.nonzero(d.any(1))[0] if d.ndim > 1 else "")
