"""Calls on fewer images than a plan was made for."""
import math

import pytest

from pat_inputs import Geometry

pytestmark = pytest.mark.gpu


def test_one_image_on_a_large_plan():
    """The interpolation of one 128^2 image costs the same on a plan for 64 images as
    on a plan for one (tiles sized for 64 take 2.5 times as long); same bits."""
    import torch
    import paper_2604_19176_amd as pat
    geom = Geometry(n=128, n_det=128, n_t=256, dt=2.0 / 256, arc_span=math.pi)
    f = torch.rand((128, 128), device="cuda")
    us, out = {}, {}
    for capacity in (1, 64):
        plan = pat.PatPlan(geom, max_batch=capacity)
        out[capacity] = plan.forward(f).clone()
        pat.pat_profile_enable(plan.handle, True)
        times = []
        for _ in range(20):
            plan.forward(f)
            times.append(pat.pat_profile_read(plan.handle, 0)[2])
        us[capacity] = 1e3 * min(times)
        plan.close()
    print("interpolation: %.1f us for one image, %.1f us on a plan for 64" % (us[1], us[64]), flush=True)
    assert torch.equal(out[1], out[64])
    assert us[64] <= 1.4 * us[1]
