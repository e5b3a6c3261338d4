"""TV gradient and value at the edges of the kernels' tiles (62 columns x 16 rows of
a workgroup, 128 x 4 of a wave), against the NumPy reference in float64.

Bounds: each quotient of magnitude at most 1 carries at most four float32 roundings,
and four of them are added with partial sums of at most 3: (4 * 4 + 3 * 3) 2^-24
absolute.  The value adds n^2 / 1024 terms per thread and a tree of ten levels.
"""

from __future__ import annotations

import numpy as np
import pytest

from oracle import tv as tvref

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [2, 3, 5, 16, 17, 61, 62, 63, 64, 65, 124, 125, 129, 257])
def test_tv_at_tile_edges(n):
    import torch
    import paper_2604_19176_amd as pat

    f = np.random.default_rng(n).standard_normal((3, n, n)).astype(np.float32)
    f[2, -1, -1] = np.inf  # reaches its neighbours' differences and nothing else
    g, tv = pat.tv_grad(torch.tensor(f, device="cuda"), 2.0 ** -7, with_value=True)
    g, tv = g.cpu().numpy(), tv.cpu().numpy()
    with np.errstate(invalid="ignore"):
        ref = np.stack([tvref.tv_grad(x.astype(np.float64), 2.0 ** -7) for x in f])
    np.testing.assert_allclose(g, ref, rtol=0, atol=25 * 2.0 ** -24, equal_nan=True)
    for b in range(2):
        want = tvref.tv_value(f[b].astype(np.float64), 2.0 ** -7)
        assert abs(tv[b] - want) <= (n * n / 1024 + 16) * 2.0 ** -24 * want
