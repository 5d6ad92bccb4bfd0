"""Variable-coefficient operator near the ends of the FP32 range: pairs of coefficients and of products are summed,
which must not overflow where the result does not."""
import numpy as np
import pytest

from tests.gpu_util import EPS, host
from tests.test_gpu_varcoef import tol_factor

pytestmark = pytest.mark.gpu
tbs = pytest.importorskip("paper_1904_03057_amd")
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("n", [1, 2, 3, 4, 5])
@pytest.mark.parametrize("cval,mval", [(3e38, 1.0), (-3e38, 1.0), (1.0, 3e38), (1e-30, 1.0)])
def test_constant_fields_near_the_range_ends(n, cval, mval):
    # splines sum to one: F(c) = m c for constant c and m without diffusion
    grid = (21, 19, 17)
    ctx = tbs.Context(grid, n, (1 / 21, 1 / 19, 1 / 17), 1e-3, "periodic")
    c = torch.full(grid[::-1], cval, dtype=torch.float32, device="cuda")
    m = torch.full_like(c, mval)
    y = torch.empty_like(c)
    ctx.apply_varcoef(c, torch.zeros_like(c), m, y)
    want = host(c[0, 0, 0]) * host(m[0, 0, 0])
    assert np.all(np.abs(host(y) / want - 1.0) <= tol_factor(n) * EPS["f32"])
