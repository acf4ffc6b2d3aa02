"""The network on grids whose layers take the convolution's variants for more
than 256 workgroups (tiles of 16 x 8 x 4 voxels times groups of 16 output
channels) with every epilogue: pooling, the concatenation read from both sources,
its split gradient, the head.  Against the oracle, with nonzero biases and
head, at the bounds of the small networks."""
import pytest

import test_gpu_denoiser as small

pytestmark = pytest.mark.gpu

# (input channels, output channels, level) of the layers with more than 24 input
# channels, and of the data gradients that split
FORWARD = [(32, 64, 2), (192, 64, 2), (96, 32, 1), (48, 16, 0)]
SPLIT = [(32, 96, 1), (64, 192, 2)]


def _groups(shape, cout, level):
    n, d, h, w = shape[0], shape[1] >> level, shape[2] >> level, shape[3] >> level
    return n * ((d + 3) // 4) * ((h + 7) // 8) * ((w + 15) // 16) * ((cout + 15) // 16)


@pytest.mark.parametrize("shape", [
    (136, 8, 8, 8),       # one tile per volume and level, mostly outside the grid
    (9, 24, 40, 72),      # two to six tiles a side, none filled at the far sides
])
def test_network_of_many_tiles(shape):
    assert all(_groups(shape, cout, level) > 256 for _, cout, level in FORWARD + SPLIT)
    small.test_network_forward_backward(shape)
