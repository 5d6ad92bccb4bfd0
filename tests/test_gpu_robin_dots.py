"""FP64 CG on Robin boxes of degree >= 2 whose sums are left to a second launch: they are added exactly as a
launch of the iteration itself with the longer z-chunks adds them, so the solve must equal, bit for
bit, the one that the z-chunk option forces into that single launch (odd and even rows: one and two
values per access; a ragged last chunk; tiles cut by both edges)."""
import numpy as np
import pytest

from tests.gpu_util import dev, host
from workloads import normal_field

pytestmark = pytest.mark.gpu
tbs = pytest.importorskip("paper_1904_03057_amd")
torch = pytest.importorskip("torch")


def chunk(grid, n):
    """Planes per chunk of the sums: about 8192 workgroups of 64 x 16 tiles, at least 4 (2n+1) planes."""
    tiles = -(-grid[0] // 64) * -(-grid[1] // 16)
    chunks = max(1, min(-(-8192 // tiles), grid[2] // (4 * (2 * n + 1))))
    return -(-grid[2] // chunks)


@pytest.mark.parametrize("n", [2, 3, 4, 5])
@pytest.mark.parametrize("grid", [(65, 33, 70), (40, 50, 61), (130, 16, 96)])
def test_sums_apart_are_bitwise_the_single_launch(n, grid):
    print("robin dots", n, grid, flush=True)
    h = (1.0 / grid[0],) * 3
    u = dev(normal_field(grid[::-1], 5))
    out = []
    for zc in (0, chunk(grid, n)):
        c = tbs.RobinContext(grid, n, h, 4.0 * h[0] ** 2, 1e-2)
        c.set_opts(zchunk=zc)
        c.ensure_workspace(tbs.PREC_FP64)
        x = torch.zeros_like(u)
        c.cg_begin(u, x, 0.0)
        rel, it = c.cg_step(25)
        rel2, it2 = c.cg_step(6)
        assert (it, it2) == (25, 31)
        out.append((host(x), rel, rel2))
    # the starting residual's sums are grouped by the plan of its own kernel: only the tolerance uses them
    assert np.array_equal(out[0][0], out[1][0])
