"""The filter's y pass at one, two and four outputs per lane (by the size of the grid),
with remainders of each, against the FP64 oracle.  Tolerance as for the filter's
other tests: sums of at most 255 x 255 FP64 products with weights of sum 1, 1e-13 of the
largest output."""

import numpy as np
import pytest

from oracle import learned as L

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("nx,ny,factor,delta", [
    (60, 509, 1, 3.0), (65, 302, 1, 20.0), (129, 701, 1, 3.0), (130, 2047, 1, 7.0), (130, 703, 1, 40.0),
    (514, 1002, 2, 8.0), (260, 1640, 4, 12.0), (48, 1604, 4, 6.0)])
def test_outputs_per_lane(nx, ny, factor, delta):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1705_09807_amd import learned as G
    print("filter", nx, ny, factor, delta, flush=True)
    r = np.random.default_rng(nx + ny)
    m = 0.05 * r.standard_normal((5, ny, nx))
    m[0] += 1.0
    out = G.filter_subsample(torch.from_numpy(m).cuda(), factor, delta).cpu().numpy()
    want = L.filtered_fields(*m, factor, delta)
    for k in range(12):
        assert np.abs(out[k] - want[k]).max() <= 1e-13 * np.abs(want[k]).max(), k
