"""The tuner against the shapes a plan or a batch comes with: no stage ends slower."""
import math

import pytest

from pat_inputs import Geometry

pytestmark = pytest.mark.gpu


def _geom(n):
    return Geometry(n=n, n_det=n, n_t=2 * n, dt=1.0 / n, arc_span=math.pi)


def _stage_us(plan, batch):
    """Kernel times of a forward and an adjoint, the least of 20."""
    import torch
    import paper_2604_19176_amd as pat
    f = torch.rand((batch,) + plan.image_shape, device="cuda")
    g = torch.rand((batch,) + plan.data_shape, device="cuda")
    pat.pat_profile_enable(plan.handle, True)
    best = [math.inf] * 10
    for _ in range(20):
        plan.forward(f)
        t = list(pat.pat_profile_read(plan.handle, 0))
        plan.adjoint(g)
        t += list(pat.pat_profile_read(plan.handle, 1))
        best = [min(a, 1e3 * b) for a, b in zip(best, t)]
    pat.pat_profile_enable(plan.handle, False)
    return best


# one 32^2 image: the default interpolation has two bands a tile (7.5 us), the lowest
# tiles listed had four (9.0); 64 images of 256^2: the default is in the lists
@pytest.mark.parametrize("n,batch", [(32, 1), (256, 64)])
def test_tuning_does_not_lose_the_defaults(n, batch):
    import paper_2604_19176_amd as pat
    plan = pat.PatPlan(_geom(n), max_batch=batch)
    before = _stage_us(plan, batch)
    plan.autotune(batch=batch)
    after = _stage_us(plan, batch)
    print("N=%d batch %d, us: %s -> %s" % (n, batch, ["%.1f" % v for v in before], ["%.1f" % v for v in after]), flush=True)
    assert after[2] <= 1.1 * before[2]  # the interpolation
    assert sum(after) <= 1.1 * sum(before)
    plan.close()


@pytest.mark.parametrize("width", [64, 128, 192, 256])
def test_the_width_a_spread_ignores_is_left_alone(width):
    """Few points: the spread's tiles have a width of their own."""
    import paper_2604_19176_amd as pat
    plan = pat.PatPlan(_geom(64))
    plan.set_launch(spr_cb=width)
    assert plan.autotune(batch=1)["spr_cb"] == width
    plan.close()


def test_entries_of_older_shape_rules_are_not_applied(tmp_path):
    """A cache entry without the version of the shape rules stays in the file, unused."""
    import json
    import re
    import paper_2604_19176_amd as pat
    cache = tmp_path / "tune.json"
    plan = pat.PatPlan(_geom(64))
    plan.autotune(batch=1, cache_path=str(cache))
    (key, entry), = json.loads(cache.read_text()).items()
    old = {re.sub(r" rules=\d+$", "", key): dict(entry, gat_cb=256, gat_th=16, gat_ib=1)}
    cache.write_text(json.dumps(old))
    again = pat.PatPlan(_geom(64))
    assert again.autotune(batch=1, cache_path=str(cache))["gat_cb"] != 256
    entries = json.loads(cache.read_text())
    assert len(entries) == 2 and set(old) < set(entries)
    plan.close()
    again.close()
