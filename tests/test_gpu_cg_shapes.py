"""Iterates of the one-kernel CG iteration in the tile shapes that the plan keeps for larger grids, against the
oracle: the tallest tiles (48 or 32 rows in FP32, 16 or 8 in FP64), which a given z-chunk length selects on any grid, and
the 32-row FP32 tiles, which the plan takes around 128^3 for degrees 1 to 3."""
import numpy as np
import pytest

from oracle import operator as op, solvers
from tests.gpu_util import dev, host, rounded
from workloads import normal_field

pytestmark = pytest.mark.gpu
tbs = pytest.importorskip("paper_1904_03057_amd")


def check(n, grid, bc, dt, zchunk, k):
    tau = 2e-3
    h = tuple(1.0 / N for N in grid)
    P = tbs.PREC_FP64 if dt == "f64" else tbs.PREC_FP32
    b = rounded(normal_field(grid[::-1], 6 + n), dt)
    ctx = tbs.Context(grid, n, h, tau, bc)
    ctx.set_opts(zchunk=zchunk)
    ctx.ensure_workspace(P)
    x = dev(np.zeros(grid[::-1]), dt)
    ctx.cg_begin(dev(b, dt), x, 0.0)
    ctx.cg_step(k - 2)
    rel, it = ctx.cg_step(2)
    xr, _, hist = solvers.cg(lambda v: op.apply(v, n, h, tau, bc), b, np.zeros_like(b), 0.0, 100, fixed_iters=k)
    assert it == k
    # the tolerances of the other iterate tests
    assert np.linalg.norm(host(x) - xr) <= (1e-10 if dt == "f64" else 1e-4) * np.linalg.norm(xr)
    assert abs(rel - hist[-1]) <= (1e-8 if dt == "f64" else 1e-3) * hist[-1]


@pytest.mark.parametrize("n", [1, 2, 3, 4, 5])
@pytest.mark.parametrize("bc", ["dirichlet", "periodic"])
@pytest.mark.parametrize("dt", ["f64", "f32"])
@pytest.mark.parametrize("grid,zchunk", [((68, 50, 24), 24), ((65, 97, 13), 5)])
def test_tallest_tiles(n, bc, dt, grid, zchunk):
    print("tall tiles", n, bc, dt, grid, zchunk, flush=True)
    check(n, grid, bc, dt, zchunk, 6)


@pytest.mark.parametrize("n", [1, 2, 3])
@pytest.mark.parametrize("bc", ["dirichlet", "periodic"])
@pytest.mark.parametrize("grid", [(128, 128, 128), (126, 125, 120), (130, 125, 118)])
def test_middle_tiles(n, bc, grid):
    print("middle tiles", n, bc, grid, flush=True)
    check(n, grid, bc, "f32", 0, 6)
