"""The adjoint spread of small launches (plans with few points times images) at
the edges of its tiles: grid sides that are no multiple of its 16 columns, row
tiles that end after one band, the periodic wrap, and batches that leave
instances of a shared tile empty.  Checked against the FP64 oracle at the
operator's parity bound, and bitwise between batched and single calls."""
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


# Ng = 32, 36, 54, 108: 2, 2.25, 3.4 and 6.75 column tiles; NB = Ng / 2 + 2 bands = 18, 20, 29, 56
@pytest.mark.parametrize("n", [16, 18, 26, 50])
@pytest.mark.parametrize("batch", [1, 3, 5])
def test_adjoint_of_small_plans(torch_dev, n, batch):
    torch = torch_dev
    import oracle
    import paper_2604_19176_amd as pat
    geom = Geometry(n=n, n_det=n + 3, n_t=2 * n + 1, dt=2.0 / (2 * n + 1), arc_span=math.radians(200.0))
    rng = np.random.default_rng(100 * n + batch)
    g = rng.standard_normal((batch, geom.n_det, geom.n_t))
    print("small spread case: N=%d batch %d" % (n, batch), flush=True)
    plan = pat.PatPlan(geom, max_batch=batch)
    gt = torch.tensor(g, dtype=torch.float32, device="cuda")
    f = plan.adjoint(gt)
    for b in range(batch):
        ref = oracle.adjoint(geom, g[b])
        err = np.linalg.norm(f[b].cpu().double().numpy() - ref) / np.linalg.norm(ref)
        assert err <= 1e-5, (b, err)
        assert torch.equal(plan.adjoint(gt[b].contiguous()), f[b])
    plan.close()
