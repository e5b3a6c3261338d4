"""The primal-dual steps over their tile shapes (rows of 64 or tiles of 16 columns, by
image side and launch size) and ragged last tiles, against the FP64 formulas; the
bound is a few float32 roundings, as in test_gpu_pdhg.py."""
import numpy as np
import pytest

from oracle import pdhg as pdref

pytestmark = pytest.mark.gpu


def _rel(a, b):
    return np.linalg.norm((a - b).ravel()) / np.linalg.norm(b.ravel())


@pytest.mark.parametrize("n,batch", [(2, 1), (15, 3), (16, 2), (17, 2), (64, 1), (65, 2), (256, 2), (272, 1), (264, 1), (272, 15)])
def test_steps_match_the_formulas(n, batch):
    import torch
    import paper_2604_19176_amd as pat
    rng = np.random.default_rng(n)
    sigma, tau, alpha = 0.3, 0.25, 0.2
    print("primal-dual case: n=%d batch %d" % (n, batch), flush=True)
    xbar, f, aty = (rng.standard_normal((batch, n, n)).astype(np.float32) for _ in range(3))
    y2 = (0.1 * rng.standard_normal((batch, n, n, 2))).astype(np.float32)
    ty2, txb, tf, taty = (torch.tensor(a, device="cuda") for a in (y2, xbar, f, aty))
    tx = torch.empty_like(tf)
    pat.pat_pd_dual_tv(ty2.data_ptr(), txb.data_ptr(), n, batch, sigma, alpha, None)
    pat.pat_pd_primal(tf.data_ptr(), tx.data_ptr(), taty.data_ptr(), ty2.data_ptr(), n, batch, tau, None)
    torch.cuda.synchronize()
    out, fn, xn = (t.cpu().double().numpy() for t in (ty2, tf, tx))
    for b in range(batch):
        dx, dy = pdref.grad(xbar[b].astype(np.float64))
        vx, vy = y2[b, ..., 0] + sigma * dx, y2[b, ..., 1] + sigma * dy
        sc = np.maximum(1.0, np.sqrt(vx * vx + vy * vy) / alpha)
        assert _rel(out[b, ..., 0], vx / sc) <= 1e-6 and _rel(out[b, ..., 1], vy / sc) <= 1e-6
        want = np.maximum(f[b] - tau * (aty[b].astype(np.float64) + pdref.grad_adjoint(out[b, ..., 0], out[b, ..., 1])), 0.0)
        assert _rel(fn[b], want) <= 1e-6 and _rel(xn[b], 2 * want - f[b]) <= 1e-6
