"""Images of an odd side: the middle pixel sits on the origin, so the transform has
no half-pixel shift.  Both operators against the FP64 oracle at the operator's
parity bound, single and batched, for a uniform arc with and without an angular
grid and for explicit detector angles; compile-time and run-time ring lengths."""
import math

import numpy as np
import pytest

from pat_inputs import Geometry

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,n_det,arc,angles", [
    (17, 16, 120.0, False), (33, 37, 250.0, False), (41, 24, 180.0, False), (75, 30, 90.0, True), (97, 32, 360.0, False)])
@pytest.mark.parametrize("batch", [1, 3])
def test_odd_sides_match_oracle(n, n_det, arc, angles, batch):
    import torch
    import oracle
    import paper_2604_19176_amd as pat
    rng = np.random.default_rng(10 * n + batch)
    th = tuple(rng.uniform(-3, 3, n_det)) if angles else None
    geom = Geometry(n=n, n_det=n_det, n_t=2 * n + 1, dt=2.0 / (2 * n + 1), arc_span=math.radians(arc), det_theta=th)
    f, g = rng.standard_normal((batch, n, n)), rng.standard_normal((batch, n_det, geom.n_t))
    print("odd side N=%d batch %d" % (n, batch), flush=True)
    plan = pat.PatPlan(geom, max_batch=batch)
    Af = plan.forward(torch.tensor(f, dtype=torch.float32, device="cuda")).cpu().double().numpy()
    Ag = plan.adjoint(torch.tensor(g, dtype=torch.float32, device="cuda")).cpu().double().numpy()
    for b in range(batch):
        for got, ref in ((Af[b], oracle.forward(geom, f[b])), (Ag[b], oracle.adjoint(geom, g[b]))):
            err = np.linalg.norm(got - ref) / np.linalg.norm(ref)
            assert err <= 1e-5, (b, err)
    plan.close()


@pytest.mark.parametrize("n,n_det", [(17, 9), (41, 16), (121, 5)])
def test_simulator_of_odd_sides(n, n_det):
    """An odd image has no centred place in an even box: the detectors lie around the
    image's centre all the same (FP64 reference with the image at the same cells)."""
    import torch
    import paper_2604_19176_amd as pat
    from oracle import simulate as ref
    geom = Geometry(n=n, n_det=n_det, n_t=35, dt=2.0 / 35, arc_span=math.radians(300.0))
    f = np.random.default_rng(n).standard_normal((n, n))
    sim = pat.PatSim(geom)
    m, h = sim.box_side, 2.0 / n
    print("odd simulator case: N=%d box %d" % (n, m), flush=True)
    assert n < m < 6 * n and m % 2 == 0
    x = -1.0 + (np.arange(n) + 0.5) * h
    off = (m - n) // 2
    box = np.zeros((m, m))
    box[off:off + n, off:off + n] = f * (x[None, :] ** 2 + x[:, None] ** 2 < geom.support_r ** 2)
    spec, kk = np.fft.fft2(box), ref.wavenumbers(m, h)
    g_ref = np.empty((n_det, geom.n_t))
    for j, t in enumerate(geom.times()):
        p = np.fft.ifft2(spec * np.cos(kk * t)).real
        for q, th in enumerate(geom.det_angles()):
            gx, gy = math.cos(th) / h + off + n / 2 - 0.5, math.sin(th) / h + off + n / 2 - 0.5
            ix, iy = math.floor(gx), math.floor(gy)
            g_ref[q, j] = ref.keys_weights(gy - iy) @ p[iy - 1:iy + 3, ix - 1:ix + 3] @ ref.keys_weights(gx - ix)
    g = sim.run(torch.tensor(f, dtype=torch.float32, device="cuda")).cpu().double().numpy()
    assert np.linalg.norm(g - g_ref) <= 1e-5 * np.linalg.norm(g_ref)
    sim.close()
