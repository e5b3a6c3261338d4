"""TV gradient and value over the kernels' launch shapes (1, 2 or 4 rows a wave by the
number of pixels, small and large images' sums), against the NumPy reference in
float64, with the bounds of test_gpu_tv_tiles.py: a quotient carries at most four
float32 roundings, four of them are added; the value adds n^2 / 1024 terms per
thread and a tree of ten levels."""
import numpy as np
import pytest

from oracle import tv as tvref

pytestmark = pytest.mark.gpu


# pixels just below and above 2^18 and 2^20
@pytest.mark.parametrize("n,batch", [(511, 1), (513, 1), (257, 4), (64, 70), (1023, 1), (1025, 1), (126, 70)])
def test_tv_by_rows_a_wave(n, batch):
    import torch
    import paper_2604_19176_amd as pat
    f = np.random.default_rng(n).standard_normal((batch, n, n)).astype(np.float32)
    print("TV case: n=%d batch %d" % (n, batch), flush=True)
    g, tv = pat.tv_grad(torch.tensor(f, device="cuda"), 2.0 ** -7, with_value=True)
    g, tv = g.cpu().numpy(), tv.cpu().numpy()
    for b in sorted({0, batch // 2, batch - 1}):
        np.testing.assert_allclose(g[b], tvref.tv_grad(f[b].astype(np.float64), 2.0 ** -7), rtol=0, atol=25 * 2.0 ** -24)
        want = tvref.tv_value(f[b].astype(np.float64), 2.0 ** -7)
        assert abs(tv[b] - want) <= (n * n / 1024 + 16) * 2.0 ** -24 * want
