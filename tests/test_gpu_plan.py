"""Automatic z-chunks of the stencil launches (one chunk per plane on small grids, uneven last chunks
on ragged ones): the operator's outputs do not depend on them, so each must equal, bit for bit, the
output with a single chunk; CG differs from it by the grouping of its FP64 sums only."""
import numpy as np
import pytest

from tests.gpu_util import dev, host
from workloads import normal_field

pytestmark = pytest.mark.gpu
tbs = pytest.importorskip("paper_1904_03057_amd")
torch = pytest.importorskip("torch")

GRIDS = [(16, 16, 16), (65, 17, 40), (130, 70, 61), (64, 200, 33)]


def _ctx(grid, n, bc, one_chunk):
    h = (1.0 / grid[0],) * 3
    tau = 4.0 * h[0] ** 2
    c = tbs.RobinContext(grid, n, h, tau, 1e-2) if bc == "robin" else tbs.Context(grid, n, h, tau, bc)
    if one_chunk:
        c.set_opts(zchunk=grid[2])
    return c


@pytest.mark.parametrize("bc", ["periodic", "dirichlet", "robin"])
@pytest.mark.parametrize("n", [1, 2, 3, 5])
@pytest.mark.parametrize("grid", GRIDS)
def test_outputs_do_not_depend_on_the_plan(bc, n, grid):
    print("plan", bc, n, grid, flush=True)
    u64, q64 = dev(normal_field(grid[::-1], 5)), dev(normal_field(grid[::-1], 6))
    out = []
    for one in (False, True):
        c = _ctx(grid, n, bc, one)
        c.ensure_workspace(-1)
        got = []
        for u, q, dt in ((u64, q64, torch.float64), (u64.float(), q64.float(), torch.float32)):
            y, b = torch.empty_like(u), torch.empty_like(u)
            c.apply(u, y)
            c.rhs(u, q, b)
            got += [y, b]
        yb = torch.empty_like(u64, dtype=torch.float32)
        c.apply(u64.to(torch.bfloat16), yb)
        r = torch.empty_like(u64)
        norms = c.residual(u64, q64, r)
        out.append((got + [yb, r], norms))
    for a, b in zip(out[0][0], out[1][0]):
        assert torch.equal(a, b)
    # the norms: sums of the same squares in another grouping
    assert np.allclose(out[0][1], out[1][1], rtol=1e-13)


@pytest.mark.parametrize("bc", ["periodic", "dirichlet", "robin"])
@pytest.mark.parametrize("prec", [tbs.PREC_FP64, tbs.PREC_MIXED])
@pytest.mark.parametrize("fused", [0, 1])
def test_steps_do_not_depend_on_the_plan(bc, prec, fused):
    grid = (65, 33, 40)
    u = dev(normal_field(grid[::-1], 7))
    out = []
    for one in (False, True):
        c = _ctx(grid, 1, bc, one)
        c.set_opts(zchunk=grid[2] if one else 0, fused_cg=fused)
        c.ensure_workspace(prec)
        x = torch.empty_like(u)
        st = c.timestep(u, None, x, prec, 1e-11, 500)
        assert st["converged"]
        out.append((host(x), st["iters"]))
    assert out[0][1] == out[1][1]
    # linear basis: A's condition number is below 100, so the rounding of the dot products stays far
    # below the tolerance the step is solved to
    assert np.linalg.norm(out[0][0] - out[1][0]) <= 1e-11 * np.linalg.norm(out[1][0])
