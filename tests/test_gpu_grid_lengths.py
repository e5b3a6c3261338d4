"""The 2D-FFT passes of compile-time grid sides, over radix mixes, tile shapes
(one sequence, a ragged last tile, the most a workgroup takes) and images at
addresses that rule out the 8-byte accesses of a column pair.  Against the FP64
oracle at the operator's parity bound; shapes and alignments bitwise."""
import math

import numpy as np
import pytest

from pat_inputs import Geometry

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch_dev():
    import torch
    assert torch.cuda.is_available()
    return torch


# grid sides 32, 48, 54, 72, 96, 144, 162, 288
@pytest.mark.parametrize("n", [16, 22, 26, 34, 48, 66, 80, 142])
def test_grid_passes(torch_dev, n):
    torch = torch_dev
    import oracle
    import paper_2604_19176_amd as pat
    geom = Geometry(n=n, n_det=12, n_t=2 * n + 5, dt=2.0 / (2 * n + 5), arc_span=math.radians(150.0))
    rng = np.random.default_rng(n)
    f, g = rng.standard_normal((n, n)), rng.standard_normal((geom.n_det, geom.n_t))
    plan = pat.PatPlan(geom)
    print("grid case: N=%d grid side %d" % (n, plan.info.n_grid), flush=True)
    ft = torch.tensor(f, dtype=torch.float32, device="cuda")
    gt = torch.tensor(g, dtype=torch.float32, device="cuda")
    Af, Ag = plan.forward(ft), plan.adjoint(gt)
    for got, ref in ((Af, oracle.forward(geom, f)), (Ag, oracle.adjoint(geom, g))):
        err = np.linalg.norm(got.cpu().double().numpy() - ref) / np.linalg.norm(ref)
        assert err <= 1e-5, err
    for shape in (dict(col_np=1, row_rpb=1), dict(col_np=3, row_rpb=5), dict(col_np=16, row_rpb=16)):
        plan.set_launch(**shape)
        assert torch.equal(plan.forward(ft), Af) and torch.equal(plan.adjoint(gt), Ag)
    buf = torch.zeros(n * n + 1, device="cuda")
    fo = buf[1:].view(n, n)
    fo.copy_(ft)
    assert torch.equal(plan.forward(fo), Af)
    assert torch.equal(plan.adjoint(gt, out=fo), Ag)
    plan.close()
