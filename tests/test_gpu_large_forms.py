"""Kernels that only large or unusual plans reach: the two-wave grid sides 1152 to
1944 and the run-time sides above 2048, heterogeneous batches with such plans, the
lane-per-column spread of heterogeneous batches, and the simulator's compile-time
boxes up to 1944 and a run-time one above 2048.  Against the 64-bit operator at the
operator's parity bound; heterogeneous batches bitwise against single calls."""
import math

import numpy as np
import pytest

from pat_inputs import Geometry

pytestmark = pytest.mark.gpu


def _check(case, seed=5):
    from perf import cases
    out, ref = cases.run(cases.prepare(case, seed)), cases.exact(case, seed)
    if not isinstance(out, tuple):
        out, ref = (out,), (ref,)
    for got, want in zip(out, ref):
        err = float((got.double() - want).norm() / want.norm())
        print("%s n=%d: %.2e" % (case["kind"], case["n"], err), flush=True)
        assert err <= 1e-5


# grid sides 324, 486, 648, 864, 972, 1152, 1296, 1458, 1536, 1728, 1944, 2304 (run-time)
@pytest.mark.parametrize("n", [160, 240, 322, 430, 486, 576, 640, 729, 760, 864, 968, 1030])
def test_grid_sides(n):
    _check(dict(kind="pair", n=n, d=16, t=200, arc=180.0, b=1, jitter=False, tmax=0.25))


# boxes 288, 324, 486, 972, 1152, 1944 and, by the run-time form, 2304
@pytest.mark.parametrize("n", [128, 144, 216, 440, 512, 864, 1024])
def test_simulator_sides(n):
    _check(dict(kind="sim", n=n, d=11, t=35, arc=300.0, b=1, jitter=False, tmax=2.0))


def _plan_io(plan, seed):
    import torch
    gen = torch.Generator(device="cuda").manual_seed(seed)
    return (torch.randn(plan.image_shape, generator=gen, device="cuda"),
            torch.randn(plan.data_shape, generator=gen, device="cuda"))


def _batch_equals_single(plans, shapes=()):
    import torch
    import paper_2604_19176_amd as pat
    batch = pat.PatBatch(plans)
    fs, gs = zip(*[_plan_io(p, i) for i, p in enumerate(plans)])
    want = [(p.forward(f).clone(), p.adjoint(g).clone()) for p, f, g in zip(plans, fs, gs)]
    for shape in (None,) + tuple(shapes):
        if shape:
            batch.set_launch(**shape)
        gb, fb = batch.forward(list(fs)), batch.adjoint(list(gs))
        for i, (g, f) in enumerate(want):
            assert torch.equal(gb[i], g) and torch.equal(fb[i], f), (shape, i)
    batch.close()
    return want, gs


def test_batch_with_sides_above_1024():
    """64^2 beside 760^2 (grid side 1536, rings up to 2048) and 1030^2 (run-time grid side)."""
    import paper_2604_19176_amd as pat
    plans = [pat.PatPlan(Geometry(n=n, n_det=d, n_t=200, dt=tmax / 200, arc_span=math.radians(arc)))
             for n, d, arc, tmax in ((64, 32, 180, 2.0), (760, 64, 270, 0.5), (1030, 16, 180, 0.25))]
    _batch_equals_single(plans[:2])   # every ring length compile-time
    _batch_equals_single(plans)
    for p in plans:
        p.close()


def test_batch_of_lane_per_column_spreads():
    """Plans of many points (here by their capacity) beside one of few, over the widths."""
    import oracle
    import paper_2604_19176_amd as pat
    geoms = [Geometry(n=40, n_det=37, n_t=75, dt=2.0 / 75, arc_span=math.radians(250.0)),
             Geometry(n=100, n_det=64, n_t=128, dt=2.0 / 128, arc_span=math.pi)]
    plans = [pat.PatPlan(geoms[0], max_batch=4096), pat.PatPlan(geoms[1], max_batch=512), pat.PatPlan(geoms[1])]
    assert all(p.info.n_points * p.max_batch > 3145728 for p in plans[:2])
    want, gs = _batch_equals_single(plans, [dict(spr_cb=w) for w in (128, 192, 256)])
    for geom, (_, f), g in zip(geoms, want, gs):
        ref = oracle.adjoint(geom, g.cpu().double().numpy())
        assert np.linalg.norm(f.cpu().double().numpy() - ref) <= 1e-5 * np.linalg.norm(ref)
    for p in plans:
        p.close()
