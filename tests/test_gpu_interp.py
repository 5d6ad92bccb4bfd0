"""Direct transform at the sizes where its line solves begin and end: lines shorter than a batch (16),
an x tile (32), the rows before the factor is constant (32) and the circulant warm-up (32 or 48), one past
each, and several; starting values other than the samples; iteration limits and non-finite values."""
import numpy as np
import pytest

from oracle import transforms as tr
from tests.gpu_util import dev, host
from workloads import normal_field

pytestmark = pytest.mark.gpu
tbs = pytest.importorskip("paper_1904_03057_amd")

GRIDS = [(5, 6, 7), (16, 17, 15), (31, 33, 32), (33, 16, 48), (65, 49, 50), (97, 5, 130), (200, 66, 5)]


@pytest.mark.parametrize("bc", ["periodic", "dirichlet"])
@pytest.mark.parametrize("n", [2, 3, 4, 5])
@pytest.mark.parametrize("grid", GRIDS)
def test_interp_line_lengths(bc, n, grid):
    print("interp", bc, n, grid, flush=True)
    s = normal_field(grid[::-1], 60 + n)
    t = tbs.Transform(grid, n, bc)
    c = dev(normal_field(grid[::-1], 70 + n))  # any start
    it, rel = t.interp(dev(s), c, rtol=1e-13, max_iter=20)
    assert rel <= 1e-13 and 1 <= it <= 2
    ref = tr.interpolate(s, n, bc)
    # error <= kappa(E) * residual, kappa(E) <= 7.5^3; the oracle's own rounding is far below
    assert np.linalg.norm(host(c) - ref) <= 450 * 1.1e-13 * np.linalg.norm(ref)


def test_interp_limits():
    grid = (20, 18, 16)
    s = normal_field(grid[::-1], 1)
    t = tbs.Transform(grid, 3, "dirichlet")
    c0 = normal_field(grid[::-1], 2)
    c = dev(c0)
    it, rel = t.interp(dev(s), c, rtol=1e-13, max_iter=0)   # nothing may change
    assert it == 0 and np.array_equal(host(c), c0) and rel > 1e-13
    it, rel = t.interp(dev(s), c, rtol=0.0, max_iter=3)     # never met: the limit is reached
    assert it == 3 and rel <= 1e-15
    it, rel = t.interp(dev(s), c, rtol=1e-18, max_iter=50)  # below rounding: ends at its level
    assert it < 50 and rel <= 1e-15
    z = dev(np.zeros(grid[::-1]))
    it, rel = t.interp(z, c, rtol=1e-13, max_iter=5)        # no samples: the start is returned
    assert it == 0
    s[3, 4, 5] = np.nan
    with pytest.raises(tbs.TbsError) as e:
        t.interp(dev(s), c, rtol=1e-13, max_iter=5)
    assert e.value.code == tbs.E_BREAKDOWN
