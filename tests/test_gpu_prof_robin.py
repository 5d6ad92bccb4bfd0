"""Kernel timing of FP64 CG on a Robin box whose iteration leaves its sums to a second launch: the record of the
iteration holds both launches."""
import pytest

from tests.gpu_util import dev
from workloads import normal_field

pytestmark = pytest.mark.gpu
tbs = pytest.importorskip("paper_1904_03057_amd")
torch = pytest.importorskip("torch")


def test_iteration_record_holds_the_sums():
    grid, n, iters = (121, 104, 90), 3, 200
    h = (1.0 / 121,) * 3
    c = tbs.RobinContext(grid, n, h, 4.0 * h[0] ** 2, 1e-3)
    c.set_opts(poll_every=0)
    c.ensure_workspace(tbs.PREC_FP64)
    b = dev(normal_field(grid[::-1], 1))
    x = torch.zeros_like(b)

    def solve():
        x.zero_()
        c.cg_begin(b, x, 0.0)
        e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        e0.record()
        c.cg_step(iters, sync=False)
        e1.record()
        e1.synchronize()
        return e0.elapsed_time(e1)

    solve()
    plain = min(solve() for _ in range(3))  # back to back, without records
    c.prof_enable()
    solve()
    ms, _, launches = c.prof_read()["cg_iter_f64"]
    assert launches == iters
    # a record around the whole iteration is no shorter than the iteration back to back; 15 % for the clocks
    assert ms >= 0.85 * plain, (ms, plain)
