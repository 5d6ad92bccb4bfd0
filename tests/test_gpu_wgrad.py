"""Weight gradients of the network's layers on the matrix cores, at the sizes where the kernel's tiles
(32 x 4 x 4 rows, one-voxel x halo of the inputs, one-row y and z halo of the gradients) begin and
end, against the FP64 oracle on the same bf16 values."""
import numpy as np
import pytest

from oracle import cnn
from oracle.rounding import to_bf16
from tests.gpu_util import host
from tests.test_gpu_net import _cl, _net
from workloads import normal_field

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

# one tile exactly, one voxel less and more along each axis, several tiles, one voxel thick, a single voxel
GRIDS = [(32, 4, 4), (31, 3, 3), (33, 5, 5), (97, 9, 6), (64, 8, 1), (1, 1, 40), (2, 1, 1), (1, 1, 1)]


@pytest.mark.parametrize("circular", [False, True])
@pytest.mark.parametrize("grid", GRIDS)
@pytest.mark.parametrize("layer", [0, 1, 3])
def test_weight_grad_tile_edges(circular, grid, layer):
    print("wgrad", circular, grid, layer, flush=True)
    ci, co = cnn.LAYERS[layer]
    net = _net(grid, training=True)
    x = to_bf16(normal_field((ci,) + grid[::-1], 80 + layer))
    g = to_bf16(normal_field((co,) + grid[::-1], 90 + layer))
    out = torch.full((co * ci * 27 + co,), float("nan"), dtype=torch.float32, device="cuda")
    net.conv_layer(layer, 2, _cl(x), _cl(g), circular, out)
    dW, db = cnn.conv3d_weight_grad(x, g, circular)
    sW, sb = cnn.conv3d_weight_grad(np.abs(x), np.abs(g), circular)
    # exact products; every partial sum is at most one FP32 rounding (2^-23, whatever its direction) of
    # the sum of absolute products, N terms, four waves and the stored result
    tol = (np.prod(grid) + 5) * 2.0 ** -23
    o = host(out)
    assert np.all(np.abs(o[:co * ci * 27] - dW.ravel()) <= tol * sW.ravel())
    assert np.all(np.abs(o[co * ci * 27:] - db) <= tol * sb)
