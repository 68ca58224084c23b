"""The backward through the projection with one view (its own kernel) and with several,
and what either does with the gradient (stored, added, applied at once), at every SH
degree and at Gaussian counts around a workgroup.

A second view that looks away adds exactly nothing, so both kernels form the same sums;
and a fused step equals the backward followed by the Adam step.  All of them share their
arithmetic in source, but each may contract products and sums differently: at most 2^-24
of the magnitudes summed per operation of a chain of under 64, so 4e-6 of a row's largest
value (and the fixed summation order, so that runs differ by nothing else)."""
import numpy as np
import pytest
import torch

import paper_2503_13086_amd as gs
import scenegen
from paper_2503_13086_amd.pipeline import DEFAULT_LR, Rasterizer

pytestmark = pytest.mark.gpu


def _scene(n, sh, sizes=((61, 45),)):
    return scenegen.small_scene(31 + n + sh, n, sh, list(sizes), log_scale_mean=-2.3)


def _away(cam):
    """The same camera turned round: it sees nothing of the scene."""
    c = dict(cam)
    turn = np.diag([-1.0, 1.0, -1.0])
    c["R"] = (turn @ np.asarray(cam["R"], np.float64)).astype(np.asarray(cam["R"]).dtype)
    c["t"] = (turn @ np.asarray(cam["t"], np.float64)).astype(np.asarray(cam["t"]).dtype)
    return c


def _run(sc, cams, mode, stride, seed=5):
    """Parameters, moments, step counters and gradient after one backward."""
    rng = np.random.default_rng(seed)
    rows = sc.params.shape[0]
    dev = lambda a: torch.as_tensor(a).cuda()
    wide = lambda a: torch.nn.functional.pad(dev(a.astype(np.float32)), (0, stride - sc.n))
    P = wide(sc.params[:, :sc.n])
    M, Vv = wide(rng.normal(0, 1e-3, (rows, sc.n))), wide(np.abs(rng.normal(0, 1e-6, (rows, sc.n))))
    base = wide(rng.normal(0, 1e-4, (rows, sc.n)))
    step = torch.nn.functional.pad(dev(rng.integers(0, 3000, sc.n).astype(np.int32)), (0, stride - sc.n))
    up = scenegen.upstream_grads(3, cams, 1e-2)
    rz = Rasterizer(0)
    try:
        gs.gs_set_backward_order(rz.ctx, gs.GS_BWD_ORDERED)
        rz.preprocess(P, sc.n, sc.sh_degree, cams)
        rz.bin_sort()
        rz.render_fwd()
        up = rz.pack_images(up)
        grad = None
        scale = [0.4] + [1.0] * (len(cams) - 1)
        if mode in ("store", "separate"):
            grad = rz.render_bwd(up, torch.full_like(P, 3.0))
        elif mode == "accumulate":
            grad = rz.render_bwd(up, base.clone(), accumulate=True)
        elif mode == "fused_grad":
            grad = torch.full_like(P, 3.0)
        if mode == "separate":
            rz.adam_step(grad, M, Vv, step, DEFAULT_LR, scale, group_mask=0b101)
        elif mode.startswith("fused"):
            rz.render_bwd_adam(up, M, Vv, step, DEFAULT_LR, scale, group_mask=0b101, grad=grad)
        torch.cuda.synchronize()
        get = lambda t: None if t is None else t[..., :sc.n].cpu().numpy().astype(np.float64)
        seen = rz.buffer(gs.GS_BUF_TOUCHED).cpu().numpy().reshape(len(cams), sc.n)
        return dict(P=get(P), m=get(M), v=get(Vv), step=get(step), grad=get(grad), base=get(base), seen=seen)
    finally:
        rz.close()


def _close(a, b, what):
    scale = np.abs(b).max(axis=-1, keepdims=True)
    assert (np.abs(a - b) <= 4e-6 * scale).all(), (what, np.max(np.abs(a - b) / np.maximum(scale, 1e-30)))


@pytest.mark.parametrize("sh", [0, 1, 2, 3])
@pytest.mark.parametrize("n", [1, 63, 255, 256, 257, 700])
def test_one_view_equals_it_beside_an_empty_one(n, sh):
    sc = _scene(n, sh)
    one = _run(sc, sc.cams, "store", n)
    two = _run(sc, [sc.cams[0], _away(sc.cams[0])], "store", n)
    assert not two["seen"][1].any() and np.array_equal(two["seen"][0], one["seen"][0])
    _close(one["grad"], two["grad"], "grad")
    assert n < 200 or np.abs(one["grad"]).max(axis=1).all()


@pytest.mark.parametrize("views", [1, 2])
@pytest.mark.parametrize("sh", [0, 1, 2, 3])
def test_what_is_done_with_the_gradient(sh, views):
    n, stride = 257, 320
    sc = _scene(n, sh, ((61, 45), (40, 52))[:views])
    sep = _run(sc, sc.cams, "separate", stride)
    acc = _run(sc, sc.cams, "accumulate", stride)
    assert (np.abs(acc["grad"] - (sep["base"] + sep["grad"])) <=
            4e-6 * (np.abs(sep["base"]).max(-1, keepdims=True) + np.abs(sep["grad"]).max(-1, keepdims=True))).all()
    for mode in ("fused", "fused_grad"):
        f = _run(sc, sc.cams, mode, stride)
        for k in ("P", "m", "v", "step"):
            _close(f[k], sep[k], (mode, k))
        if mode == "fused_grad":
            _close(f["grad"], sep["grad"], "written gradient")


@pytest.mark.parametrize("views", [1, 2])
def test_parameters_larger_than_the_cache(views):
    """Past 256 MB the fused step stores the parameters another way (stride alone
    decides)."""
    n, stride = 257, (1 << 28) // (59 * 4) + 64
    sc = _scene(n, 3, ((61, 45), (40, 52))[:views])
    small, big = (_run(sc, sc.cams, "fused", s) for s in (n, stride))
    for k in ("P", "m", "v", "step"):
        assert np.array_equal(small[k], big[k]), k
