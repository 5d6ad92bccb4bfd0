"""Variable-coefficient operator where its strips (64 - 2n columns, 16 rows in FP32 and 8 in FP64) and
z-chunks begin and end: one strip exactly, one column, row and plane more, and the smallest grids."""
import numpy as np
import pytest

from oracle import varcoef
from tests.gpu_util import EPS, dev, host, rounded
from tests.test_gpu_varcoef import abs_scale, coef_fields, tol_factor
from workloads import normal_field

pytestmark = pytest.mark.gpu
tbs = pytest.importorskip("paper_1904_03057_amd")
torch = pytest.importorskip("torch")

CASES = [(n, bc, g) for n in (1, 2, 3, 5) for bc in ("dirichlet", "periodic")
         for g in ((64 - 2 * n, 16, 11), (65 - 2 * n, 17, 12), (2 * n + 1, 2 * n + 1, 2 * n + 1))]


@pytest.mark.parametrize("n,bc,grid", CASES)
@pytest.mark.parametrize("dt", ["f64", "f32"])
def test_strip_edges_match_oracle(n, bc, grid, dt, monkeypatch):
    print("varcoef tiles", n, bc, grid, dt, flush=True)
    shape = grid[::-1]
    h, tau = (1 / 21, 1 / 19, 1 / 18), 2e-3
    c = rounded(normal_field(shape, 30 + n), dt)
    d, m = (rounded(v, dt) for v in coef_fields(shape, 40 + n, tau))
    ctx = tbs.Context(grid, n, h, tau, bc)
    y = torch.full(shape, float("nan"), dtype=torch.float64 if dt == "f64" else torch.float32, device="cuda")
    ctx.apply_varcoef(dev(c, dt), dev(d, dt), dev(m, dt), y)
    ref = varcoef.apply(c, d, m, n, h, bc)
    scale = abs_scale(c, d, m, n, h, bc, monkeypatch)
    # rounding bound of one output's longest chain, as for the other parity tests of the operator
    tol = tol_factor(n) * EPS[dt] * scale + (np.abs(ref) * EPS[dt] if dt == "f32" else 0.0)
    assert np.all(np.abs(host(y) - ref) <= tol)
