"""Direct transform of samples whose norm vanishes: zero samples have zero coefficients whatever the start, and
samples whose squares underflow are solved like any others."""
import numpy as np
import pytest

from oracle import transforms as tr
from tests.gpu_util import dev, host
from workloads import normal_field

pytestmark = pytest.mark.gpu
tbs = pytest.importorskip("paper_1904_03057_amd")

GRID = (20, 18, 16)


@pytest.mark.parametrize("bc", ["periodic", "dirichlet"])
def test_zero_samples_give_zero_coefficients(bc):
    t = tbs.Transform(GRID, 3, bc)
    z = dev(np.zeros(GRID[::-1]))
    c = dev(normal_field(GRID[::-1], 2))
    it, rel = t.interp(z, c, rtol=1e-13, max_iter=5)
    assert rel == 0.0 and not host(c).any()
    c0 = normal_field(GRID[::-1], 2)
    c = dev(c0)
    it, rel = t.interp(z, c, rtol=1e-13, max_iter=0)  # no step allowed: the start, and its residual
    assert it == 0 and np.array_equal(host(c), c0) and rel > 0.0
    c = dev(np.zeros(GRID[::-1]))
    assert t.interp(z, c, rtol=1e-13, max_iter=0) == (0, 0.0)


@pytest.mark.parametrize("mag", [1e-170, 1e-250])
def test_samples_whose_squares_underflow(mag):
    s = normal_field(GRID[::-1], 1)
    t = tbs.Transform(GRID, 3, "dirichlet")
    c = dev(s * mag)
    it, rel = t.interp(dev(s * mag), c, rtol=1e-13, max_iter=5)
    assert rel <= 1e-13 and it >= 1
    ref = tr.interpolate(s, 3, "dirichlet")
    # error <= kappa(E) * residual, kappa(E) = 27 for cubic splines
    assert np.linalg.norm(host(c) / mag - ref) <= 27 * 1.1e-13 * np.linalg.norm(ref)
