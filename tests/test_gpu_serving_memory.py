"""What the serving engine's admission charges for a view's pixels covers what a step holds
for them, with no more than a third to spare: a job that fits is not turned away."""
import numpy as np
import pytest
import torch

import scenegen

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("jobs", [1, 3])
def test_pixel_charge(jobs):
    from paper_2503_13086_amd.serving import Engine, Field
    n, (w, h) = 600, (1296, 864)
    sc = scenegen.small_scene(19, n, 3, [(w, h)] * jobs, log_scale_mean=-6.0)   # few pairs: pixels are all there is
    eng = Engine(Field(sc.params[:, :n - jobs], 3, capacity=n), max_slots=jobs, t_i=8, w_l1=0.47, w_dssim=0.12,
                 w_load=0.41)
    eng.pairs_per_view = 0
    try:
        px, active = w * h, []
        for i in range(jobs):
            t = torch.rand(3 * px, device="cuda")
            block = torch.as_tensor(np.ascontiguousarray(sc.params[:, n - jobs + i: n - jobs + i + 1]))
            active.append(eng.register(sc.cams[i], t, [0.5] * i, block))
        base = eng.rz.memory_bytes()
        eng.step(active)
        torch.cuda.synchronize()
        held = eng.rz.memory_bytes() - base + eng._img.numel() * 8 + (12 * px * jobs if jobs > 1 else 0)
        charged = jobs * (eng._view_bytes(n, px) - eng._view_bytes(n, 0))
        small = jobs * eng._view_bytes(n, 0)        # everything that does not go with the pixels
        print(f"held {held / px / jobs:.1f} B per pixel (up to {small / px / jobs:.1f} of it for other things), "
              f"charged {charged / px / jobs:.1f}", flush=True)
        assert held - small <= charged <= 4 / 3 * held
    finally:
        eng.close()
