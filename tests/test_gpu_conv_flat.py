"""Convolutions of one z plane on more than 256 tiles (blocks of 64 x 8 x 1
voxels): forward and data gradient against the oracle at the bound of the other
grids, sides one past and one short of a block, rows of one voxel, output
channels that do not fill the last 16 or 32."""
import pytest

import test_gpu_denoiser as volumes

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("cin,cout,shape", [
    (16, 16, (1, 1, 129, 257)),
    (40, 24, (1, 1, 127, 319)),
    (8, 48, (3, 1, 65, 191)),
    (32, 32, (1, 1, 1, 4111)),
    (24, 16, (7, 1, 150, 17)),    # the narrowest
])
def test_conv_of_one_plane(cin, cout, shape):
    n, _, h, w = shape
    assert n * ((h + 7) // 8) * ((w + 15) // 16) * ((cout + 15) // 16) > 256
    volumes.test_conv_forward_and_data_gradient_many_tiles(cin, cout, shape)
