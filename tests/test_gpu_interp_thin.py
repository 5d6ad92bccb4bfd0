"""Direct transform of thin boxes, whose few long lines are cut into segments: against the oracle where the
segments (256 samples and more, 32 or 48 of lead-in) begin and end, and no slower than CG on the same operator."""
import numpy as np
import pytest

from oracle import transforms as tr
from tests.gpu_util import dev, host
from workloads import normal_field

pytestmark = pytest.mark.gpu
tbs = pytest.importorskip("paper_1904_03057_amd")
torch = pytest.importorskip("torch")

LONG = [511, 512, 513, 575, 769, 2049]


@pytest.mark.parametrize("bc", ["periodic", "dirichlet"])
@pytest.mark.parametrize("n", [2, 3, 4, 5])
@pytest.mark.parametrize("axis", [0, 1, 2])
def test_segment_edges(bc, n, axis):
    for length in LONG:
        grid = [5, 7, 6]
        grid[axis] = length
        print("thin", bc, n, grid, flush=True)
        s = normal_field(grid[::-1], 60 + n)
        t = tbs.Transform(grid, n, bc)
        c = dev(normal_field(grid[::-1], 70 + n))
        it, rel = t.interp(dev(s), c, rtol=1e-13, max_iter=20)
        assert rel <= 1e-13 and 1 <= it <= 2
        ref = tr.interpolate(s, n, bc)
        # error <= kappa(E) * residual, kappa(E) <= 7.5^3; the oracle's own rounding is far below
        assert np.linalg.norm(host(c) - ref) <= 450 * 1.1e-13 * np.linalg.norm(ref)


@pytest.mark.parametrize("axis", [0, 1, 2])
def test_no_slower_than_cg(axis):
    grid = [5, 5, 5]
    grid[axis] = 1 << 19
    s = dev(np.random.default_rng(1).standard_normal(grid[::-1]))
    t = tbs.Transform(grid, 3, "dirichlet")
    t.ensure_workspace(tbs.PREC_FP64)
    c = torch.empty_like(s)

    def best(f):
        times = []
        for _ in range(4):
            c.copy_(s)
            e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            e0.record()
            f()
            e1.record()
            e1.synchronize()
            times.append(e0.elapsed_time(e1))
        return min(times)

    def cg():
        t.cg_begin(s, c, 1e-12)
        assert t.cg_step(1000)[0] <= 1e-12

    solve = best(lambda: t.interp(s, c, 1e-12, 1000))
    assert solve <= best(cg)
