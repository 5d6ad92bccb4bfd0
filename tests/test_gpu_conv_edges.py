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


@pytest.mark.parametrize("circular", [False, True])
@pytest.mark.parametrize("grid", GRIDS + [(161, 130, 70)])   # the last: chunks of several planes, ragged
def test_last_layer_tile_edges(circular, grid):
    print("last layer", circular, grid, flush=True)
    theta = cnn_init(7)
    theta[cnn.N_PARAMS - 1] = 0.25
    net = _net(grid, theta=theta)
    W = cnn.unpack(to_bf16(theta))[3][0]
    x = to_bf16(normal_field((16,) + grid[::-1], 70))
    out = torch.full(grid[::-1] + (1,), float("nan"), dtype=torch.float32, device="cuda")
    net.conv_layer(3, 0, _cl(x), None, circular, out)
    ref = cnn.conv3d(x, W, np.array([0.25]), circular)
    # exact products, 432 of them, the bias and their roundings in FP32
    tol = 433 * 2.0 ** -23 * (cnn.conv3d(np.abs(x), np.abs(W), None, circular) + 0.25)
    assert np.all(np.abs(_from_cl(out) - ref) <= tol)


def test_last_layer_keeps_an_infinity_to_its_stencil():
    grid = (40, 12, 9)
    net = _net(grid, theta=cnn_init(7))
    x = to_bf16(normal_field((16,) + grid[::-1], 71))
    x[3, 4, 5, 17] = np.inf
    out = torch.empty(grid[::-1] + (1,), dtype=torch.float32, device="cuda")
    net.conv_layer(3, 0, _cl(x), None, False, out)
    bad = ~np.isfinite(host(out)[..., 0])
    near = np.zeros_like(bad)
    near[3:6, 4:7, 16:19] = True
    assert np.array_equal(bad, near)
