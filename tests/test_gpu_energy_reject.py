"""Energy test of the learned guess (guess_test = 1), rejected guess: the step goes on from the plain guess's
residual and its sums, so it takes the sweeps, iterations and values of a step without a network, also
where the network's output is not finite."""
import numpy as np
import pytest

from oracle import cnn
from tests.gpu_util import dev, host
from workloads import cnn_init, normal_field

pytestmark = pytest.mark.gpu
tbs = pytest.importorskip("paper_1904_03057_amd")


@pytest.mark.parametrize("output", ["zero", "infinite"])
@pytest.mark.parametrize("prec", [tbs.PREC_MIXED, tbs.PREC_MIXED_BF16])
def test_rejected_guess_leaves_the_plain_step(output, prec):
    grid, n, tau = (32, 24, 20), 3, 1e-3
    h = tuple(1.0 / (N + 1) for N in grid)
    u = dev(normal_field(grid[::-1], 3))
    theta = np.zeros(cnn.N_PARAMS, dtype=np.float32) if output == "zero" else cnn_init(1)
    theta[cnn.N_PARAMS - 1] = 0.0 if output == "zero" else 1.0
    net = tbs.Net()
    net.ensure_workspace(grid, 1, False)
    net.set_weights(theta)
    net.set_hparams(out_scale=1.0 if output == "zero" else 1e45)
    ctx = tbs.Context(grid, n, h, tau, "dirichlet")
    ctx.set_opts(guess_test=1)
    ctx.ensure_workspace(prec)
    a, b = dev(np.zeros(grid[::-1])), dev(np.zeros(grid[::-1]))
    s0 = ctx.timestep(u, None, b, prec, 1e-8, 500, None)
    s1 = ctx.timestep(u, None, a, prec, 1e-8, 500, net)
    assert s1["used_learned_guess"] == 0 and s1["converged"]
    for k in ("sweeps", "iters", "rel_res_plain", "rel_res_fp64"):
        assert s1[k] == s0[k], k
    assert np.array_equal(host(a), host(b))
