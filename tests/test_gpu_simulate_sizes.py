"""The simulator's two forms (compile-time and run-time box sides) where one
gives way to the other."""
import math

import pytest

from pat_inputs import Geometry

pytestmark = pytest.mark.gpu


def _run_us(n):
    """Microseconds of one run on an n^2 image, 256 detectors, 512 samples."""
    import torch
    import paper_2604_19176_amd as pat
    sim = pat.PatSim(Geometry(n=n, n_det=256, n_t=512, dt=2.0 / 512, arc_span=math.radians(270)))
    f, out = torch.rand((n, n), device="cuda"), torch.empty((256, 512), device="cuda")
    for _ in range(3):
        sim.run(f, out=out)
    best = math.inf
    for _ in range(5):
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record()
        for _ in range(20):
            sim.run(f, out=out)
        b.record()
        b.synchronize()
        best = min(best, a.elapsed_time(b) * 1e3 / 20)
    print("simulator n=%d box %d: %.1f us" % (n, sim.box_side, best), flush=True)
    return best


def test_small_boxes_take_the_short_form():
    """A 54^2 box has a sixteenth of a 216^2 box's cells; 0.61 of its time by the
    run-time form, 0.88 by the compile-time form, whose columns are four lanes."""
    assert _run_us(24) <= 0.75 * _run_us(96)
