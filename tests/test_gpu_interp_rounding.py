"""Direct transform asked for less than rounding allows: it ends at the rounding level of the residual, also for
samples that alternate in sign, whose coefficients are up to 400 times larger (degree 5)."""
import numpy as np
import pytest

from tests.gpu_util import dev, host

pytestmark = pytest.mark.gpu
tbs = pytest.importorskip("paper_1904_03057_amd")


@pytest.mark.parametrize("bc", ["periodic", "dirichlet"])
@pytest.mark.parametrize("n", [3, 4, 5])
@pytest.mark.parametrize("rtol", [1e-14, 1e-16])
def test_alternating_samples_end_at_rounding(bc, n, rtol):
    grid = (48, 36, 24)
    z, y, x = np.indices(grid[::-1])
    s = (-1.0) ** (x + y + z) * np.random.default_rng(n).uniform(0.98, 1.02, grid[::-1])
    t = tbs.Transform(grid, n, bc)
    c = dev(s)
    it, rel = t.interp(dev(s), c, rtol=rtol, max_iter=40)
    assert it < 40
    # E c: three passes of 2 floor(n/2) + 1 positive taps that sum to one, and the subtraction
    k = 3 * (2 * (n // 2) + 1) + 1
    assert rel <= k * 2.0 ** -53 * (1 + np.linalg.norm(host(c)) / np.linalg.norm(s))


@pytest.mark.parametrize("bc", ["periodic", "dirichlet"])
def test_rounding_level_needs_no_further_solve(bc):
    # the level is a few 1e-15 to 1e-14 of the samples here, and where it lies must not decide: the second solve
    # reduces nothing any more
    grid = (33, 41, 29)
    z, y, x = np.indices(grid[::-1])
    t = tbs.Transform(grid, 5, bc)
    for v in np.random.default_rng(0).uniform(0.5, 1.0, 304):
        s = dev((-1.0) ** (x + y + z) * v)
        c = s.clone()
        it, _ = t.interp(s, c, rtol=1e-17, max_iter=40)
        assert it <= 2
