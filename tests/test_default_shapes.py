"""The launch shapes plan creation picks, over every grid side of images up to
1024^2 and batches that select each column tile: never one the plan refuses."""
import ctypes
import math

import pytest

from pat_inputs import Geometry


def _grid_side(n):
    return min(p for p in (2 ** a * 3 ** b for a in range(1, 13) for b in range(8)) if p >= 2 * n)


# the smallest and the largest image of every grid side
SIDES = {}
for _n in range(18, 1025):
    SIDES.setdefault(_grid_side(_n), []).append(_n)
IMAGES = sorted({v for ns in SIDES.values() for v in (ns[0], ns[-1])})


@pytest.mark.parametrize("batch", [1, 4, 5, 6, 8, 64])
def test_every_image_size_has_default_shapes(batch):
    """Plan creation derives tables and shapes on the host before it touches the
    device: without a GPU it ends in a HIP or allocation error, never UNSUPPORTED."""
    import paper_2604_19176_amd as pat
    from paper_2604_19176_amd import _lib
    lib = _lib.load()
    refused = []
    for n in IMAGES:
        desc = pat.desc_from_geometry(Geometry(n=n, n_det=4, n_t=16, dt=0.05 / 16, arc_span=math.pi), max_batch=batch)
        out = ctypes.c_void_p()
        rc = lib.pat_plan_create(ctypes.byref(desc), ctypes.byref(out))
        if rc == 0:
            lib.pat_plan_destroy(out)
        elif rc == _lib.PAT_ERR_UNSUPPORTED:
            refused.append(n)
    assert not refused, refused


# grid sides 1728 and 1944, where eight pairs are more than a workgroup may be asked for
@pytest.mark.gpu
@pytest.mark.parametrize("n", [770, 900])
def test_wide_grid_batches(n):
    import torch
    from perf import cases
    case = dict(kind="pair", n=n, d=9, t=64, arc=200.0, b=6, jitter=False, tmax=0.25)
    print("batch of 6 at N=%d" % n, flush=True)
    out = cases.run(cases.prepare(case, 5))
    for got, ref in zip(out, cases.exact(case, 5)):
        for b in range(6):
            assert float((got[b].double() - ref[b]).norm() / ref[b].norm()) <= 1e-5
    torch.cuda.synchronize()
