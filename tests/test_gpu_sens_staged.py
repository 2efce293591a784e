"""Exactness of the prediction that keeps one bit per element of a region's footprint: planes of any size (rows below
and above a machine word, pieces that start before or end behind a channel's run, the end of the tensor), thresholds on
both sides of the zero border, and seeds over which the lowest bits of the draw's argument carry and do not carry."""
import numpy as np
import pytest

from test_gpu_sensitivity import _predict_both
from util import from_vals, stored

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("N,C,H,W,k,stride,pad,x,y", [
    (1, 1, 1, 1, 1, 1, 0, 1, 0), (3, 5, 7, 7, 3, 1, 1, 7, 0), (2, 3, 13, 13, 3, 1, 1, 4, 9), (2, 4, 5, 40, 5, 1, 2, 40, 0),
    (1, 3, 6, 65, 3, 1, 1, 20, 0), (2, 7, 19, 3, 3, 2, 1, 5, 0), (2, 64, 27, 27, 3, 1, 1, 54, 288)])
@pytest.mark.parametrize("thr", [-0.2, 0.4])
def test_odd_planes_and_thresholds(dtype, N, C, H, W, k, stride, pad, x, y, thr):
    print("prediction", dtype, N, C, H, W, k, stride, pad, x, y, thr, flush=True)
    rng = np.random.default_rng(H * W + C)
    Av = stored(rng.standard_normal((N, C, H, W)), dtype)
    for seed in (1, 123456789, 2 ** 63 + 5):
        _predict_both(Av, from_vals(Av, dtype), k, stride, pad, x, y, 300, 500, thr, seed, seed % 7)


@pytest.mark.parametrize("N,C,H,W,k,stride,pad,x,y,permille", [
    (2, 3, 5, 30, 3, 1, 1, 30, 27, 300), (2, 2, 4, 31, 3, 1, 1, 31, 0, 300), (1, 2, 4, 62, 3, 1, 1, 62, 0, 1000), (1, 2, 4, 63, 3, 1, 1, 7, 0, 500),
    (3, 1, 3, 33, 1, 1, 0, 33, 0, 1000), (1, 5, 9, 9, 3, 1, 1, 1, 0, 1), (1, 4, 16, 16, 3, 1, 1, 256, 0, 1000), (2, 30, 9, 13, 3, 1, 1, 13, 54, 900)])
def test_words_of_a_row_and_shares_of_a_band(N, C, H, W, k, stride, pad, x, y, permille):
    """Bordered rows of exactly one and two words and one element more, odd first elements, the words at the tensor's end; bands
    of one draw, of whole and part rounds of 256 draws, and of more than 64 rounds; one band and many per workgroup."""
    print("prediction, words", N, C, H, W, k, x, y, permille, flush=True)
    rng = np.random.default_rng(H * W + C)
    for dtype in ("bf16", "f32"):
        Av = stored(rng.standard_normal((N, C, H, W)), dtype)
        for seed, thr in ((11, 0.1), (2 ** 61 + 3, -0.3)):
            _predict_both(Av, from_vals(Av, dtype), k, stride, pad, x, y, permille, 500, thr, seed, 2)


@pytest.mark.parametrize("N,C,H,W,k,stride,pad,x,y,permille", [
    (300, 2, 13, 13, 3, 1, 1, 4, 0, 300), (70, 4, 14, 14, 3, 1, 1, 14, 0, 300), (40, 6, 13, 13, 3, 1, 1, 5, 27, 400), (120, 3, 9, 40, 3, 2, 1, 7, 0, 500),
    (257, 1, 8, 8, 1, 1, 0, 3, 0, 1000), (300, 96, 240, 4, 3, 1, 1, 4, 0, 1), (1, 910, 188, 98, 3, 1, 1, 1, 0, 1)])
def test_several_bands_of_a_workgroup(N, C, H, W, k, stride, pad, x, y, permille):
    """Images enough that workgroups take several bands, the last one fewer, in rows of one and two words and with two column
    blocks; an image of which not all bands fit, and one of which a single band takes more LDS than is allotted."""
    print("prediction, bands", N, C, H, W, k, stride, x, y, permille, flush=True)
    rng = np.random.default_rng(H * W + C)
    for dtype in ("bf16", "f32") if N * C * H * W < 1 << 20 else ("bf16",):
        Av = stored(rng.standard_normal((N, C, H, W), dtype=np.float32), dtype)
        _predict_both(Av, from_vals(Av, dtype), k, stride, pad, x, y, permille, 500, 0.1, 2 ** 40 + 9, 3)
