"""The simulator's compile-time box sides over the radix mixes of their first
pass (odd and even radices, several rounds per lane), with detector rows that are
mostly unread (few detectors) and a ragged last chunk of sample pairs.  Against
the FP64 reference at the simulator's tolerance."""
import math

import numpy as np
import pytest

from pat_inputs import Geometry, make_phantom

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch_dev():
    import torch
    assert torch.cuda.is_available()
    return torch


# boxes 36, 54, 72, 162, 216; 1 to 37 detectors
@pytest.mark.parametrize("n,n_det", [(16, 1), (26, 3), (32, 37), (74, 5), (96, 16)])
def test_simulator_boxes(torch_dev, n, n_det):
    torch = torch_dev
    import paper_2604_19176_amd as pat
    from oracle import simulate as ref
    geom = Geometry(n=n, n_det=n_det, n_t=35, dt=2.0 / 35, arc_span=math.radians(300))
    f = make_phantom(n, 5, 2, 1, 7)
    sim = pat.PatSim(geom)
    print("simulator case: n=%d D=%d box %d" % (n, n_det, sim.box_side), flush=True)
    g = sim.run(torch.tensor(f, dtype=torch.float32, device="cuda")).cpu().double().numpy()
    g_ref = ref.simulate(geom, f)
    assert np.linalg.norm(g - g_ref) <= 1e-5 * np.linalg.norm(g_ref)
