"""The network's convolutions at the sizes where their tiles (32 x 8 columns of a chunk of planes, 16-voxel
rows, one-voxel halo) begin and end, against the FP64 oracle on the same bf16 values."""
import numpy as np
import pytest

from oracle import cnn
from oracle.rounding import to_bf16
from tests.gpu_util import host
from tests.test_gpu_net import _cl, _from_cl, _net
from workloads import cnn_init, normal_field

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

# one tile exactly, one voxel less and more along each axis, several tiles, one voxel thick, a single voxel
GRIDS = [(32, 8, 4), (31, 7, 3), (33, 9, 5), (97, 17, 6), (64, 8, 1), (1, 1, 40), (2, 1, 1), (1, 1, 1)]


@pytest.mark.parametrize("circular", [False, True])
@pytest.mark.parametrize("grid", GRIDS)
@pytest.mark.parametrize("layer", [1, 3])
def test_data_grad_tile_edges(circular, grid, layer):
    print("dgrad", circular, grid, layer, flush=True)
    ci, co = cnn.LAYERS[layer]
    theta = cnn_init(8)
    net = _net(grid, theta=theta)
    W = cnn.unpack(to_bf16(theta))[layer][0]
    g = to_bf16(normal_field((co,) + grid[::-1], 60 + layer))
    out = torch.full(grid[::-1] + (ci,), float("nan"), dtype=torch.float32, device="cuda")
    net.conv_layer(layer, 1, None, _cl(g), circular, out)
    ref = cnn.conv3d_data_grad(g, W, circular)
    # exact products, 27 co of them and their roundings in FP32
    tol = 27 * co * 2.0 ** -23 * cnn.conv3d_data_grad(np.abs(g), np.abs(W), circular)
    assert np.all(np.abs(_from_cl(out) - ref) <= tol)
