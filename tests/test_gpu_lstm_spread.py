"""GPU parity of what surrounds an LSTM layer's recurrences: gathers of every second to fifth unit from addresses of either parity,
input gradients whose rows end in the middle of a 16-byte piece, and weight gradients added from partial sums."""
import numpy as np
import pytest

from oracle import patterns as P
from paper_2203_05705_amd import binding as ard
from test_gpu_lstm import _check
from util import from_vals, stored

pytestmark = pytest.mark.gpu


def _case(dtype, T, B, I, H, dp, b, scale):
    rng = np.random.default_rng(T * 100 + H + dp)
    x = stored(rng.standard_normal((T, B, I)), dtype)
    W = stored(rng.uniform(-scale, scale, (4 * H, I + H)), dtype)
    dh = stored(rng.standard_normal((T, B, H)), dtype)
    _check(dtype, x, W, dh, P.row_mask(H, dp, b), ard.Pattern.row(dp, b), from_vals(x, dtype), from_vals(W, dtype), from_vals(dh, dtype),
           f"lstm {dtype} T={T} B={B} I={I} H={H} dp={dp} b={b}")


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("dp", [1, 2, 3, 4, 5])
@pytest.mark.parametrize("I,H", [(37, 83), (46, 96), (24, 129)])
def test_gathers(dtype, I, H, dp):
    _case(dtype, 3, 5, I, H, dp, dp, 0.2)


@pytest.mark.parametrize("T,B,I,H,dp,b", [(64, 128, 1004, 998, 2, 1), (48, 128, 520, 1533, 3, 2)])
def test_weight_gradients_from_partial_sums(T, B, I, H, dp, b):
    _case("bf16", T, B, I, H, dp, b, 0.03)
