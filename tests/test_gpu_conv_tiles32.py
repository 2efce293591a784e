"""GPU parity of the fp32 convolutions on every tile they choose, asserted case by case: rows and pixels left over, output rows in whole
groups of four pixels (which leave from the registers of the tiles along the pixels) and not, all maps kept and a list of them."""
import pytest

import dryrun as D
import test_gpu_conv_planes as planes

pytestmark = pytest.mark.gpu


def _tile(mode, N, C, Cout, S, k, rate):
    with D.dry_run() as lib:
        D.launches(lib)
        assert D.conv_calls(lib, D.FakeHeap(), D.F32, N, C, Cout, S, S, k, 1, k // 2, C - int(rate * C), modes=(mode,)) == [0]
        return [i for i in D.instances(lib) if i.startswith("gemm_f32_kernel")]


@pytest.mark.parametrize("mode,tile,N,C,Cout,S,k,rate", [
    (1, "32, 128", 11, 11, 127, 20, 3, 0.0), (1, "32, 128", 52, 16, 9, 20, 1, 0.0), (1, "32, 128", 60, 19, 143, 18, 1, 0.0), (2, "32, 128", 41, 37, 18, 20, 3, 0.5),
    (1, "32, 256", 16, 50, 129, 28, 1, 0.0), (1, "64, 128", 41, 68, 111, 18, 1, 0.0), (1, "64, 256", 30, 9, 73, 28, 3, 0.0), (1, "128, 128", 34, 84, 116, 27, 1, 0.0),
    (1, "64, 64", 52, 51, 36, 13, 3, 0.0), (1, "32, 32", 37, 88, 137, 9, 1, 0.0), (1, "32, 32", 7, 120, 181, 16, 1, 0.0), (1, "16, 16", 2, 72, 96, 13, 3, 0.0)])
def test_every_tile(mode, tile, N, C, Cout, S, k, rate):
    assert _tile(mode, N, C, Cout, S, k, rate) == [f"gemm_f32_kernel<{tile}, 1>"]
    planes.test_planes(N, C, Cout, S, S, k, k // 2, rate)
