"""GPU parity of the fp32 convolutions' tiles that lie along the pixels: 256 and 128 pixels by 64 and 32 channels, with rows and pixels
left over, pixels in whole groups of four (which leave from the registers) and not, all maps kept and a list of them."""
import pytest

import test_gpu_conv_planes as planes

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,C,Cout,S,k,rate", [(20, 64, 90, 27, 3, 0.0), (8, 100, 40, 56, 3, 0.5), (64, 64, 64, 32, 3, 0.5), (9, 70, 33, 28, 3, 0.3),
                                               (37, 20, 100, 16, 3, 0.0), (16, 24, 130, 28, 5, 0.5), (5, 18, 17, 12, 3, 0.0)])
def test_tiles_along_the_pixels(N, C, Cout, S, k, rate):
    planes.test_planes(N, C, Cout, S, S, k, k // 2, rate)
