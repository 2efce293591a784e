"""GPU parity of the fp32 LSTM whose steps are one launch each: kept units around its tiles of 16 and its half slices of 8, batch
rows around 16, contractions of one slice up to more than four per wavefront, every group of dropped units a tile can own, one step,
and the first layers beyond its range (which take two launches a step)."""
import numpy as np
import pytest

from dryrun import FakeHeap, dry_run, launches, lstm_calls
from oracle import patterns as P
from paper_2203_05705_amd import binding as ard
from test_gpu_lstm import _check
from util import from_vals, stored


@pytest.mark.gpu
@pytest.mark.parametrize("T,B,I,H,dp,b", [(3, 1, 5, 1, 1, 1), (2, 15, 8, 8, 1, 1), (4, 17, 20, 9, 1, 1), (1, 16, 16, 40, 3, 2), (5, 16, 33, 47, 2, 1), (3, 33, 24, 70, 3, 3),
                                          (4, 5, 16, 137, 1, 1), (3, 40, 16, 301, 4, 4), (2, 20, 30, 530, 1, 1), (3, 8, 12, 1100, 2, 2), (2, 3, 16, 700, 8, 5),
                                          (2, 70, 8, 648, 1, 1), (2, 70, 8, 650, 1, 1), (3, 20, 16, 300, 8, 3), (3, 20, 16, 100, 6, 2)])
def test_one_launch_steps(T, B, I, H, dp, b):
    print("lstm f32 steps", T, B, I, H, dp, b, flush=True)
    rng = np.random.default_rng(T * 1000 + H)
    x = stored(rng.standard_normal((T, B, I)), "f32")
    lim = 1.0 / np.sqrt(H)
    W = stored(rng.uniform(-lim, lim, (4 * H, I + H)), "f32")
    dh = stored(rng.standard_normal((T, B, H)), "f32")
    _check("f32", x, W, dh, P.row_mask(H, dp, b), ard.Pattern.row(dp, b), from_vals(x, "f32"), from_vals(W, "f32"), from_vals(dh, "f32"), "lstm f32")


def test_which_layers_take_them():
    with dry_run() as lib:
        for B, H, one in ((20, 128, True), (70, 647, True), (70, 648, False), (128, 1024, False)):
            launches(lib)
            assert lstm_calls(lib, FakeHeap(), ard.F32, 4, B, 32, H, None) == [0, 0]
            _, names = launches(lib)
            assert (names.count("lstm_step32_fwd_kernel"), names.count("lstm_step32_bwd_kernel")) == ((4, 4) if one else (0, 0))
            assert any(n.startswith("lstm_cell") for n in names) != one


def test_which_forward_passes_write_too_many_zeros_for_them():
    """Every eighth unit kept (not yet every sixth): full tiles of 16 rows and units take two launches a step, and so does a single step."""
    with dry_run() as lib:
        for T, B, H, dp, one in ((4, 8, 626, 8, True), (4, 38, 894, 8, False), (4, 25, 160, 6, True), (4, 40, 64, 8, True), (4, 38, 894, 4, True), (1, 8, 64, 2, False)):
            launches(lib)
            assert lstm_calls(lib, FakeHeap(), ard.F32, T, B, 32, H, (dp, 1)) == [0, 0]
            _, names = launches(lib)
            assert (names.count("lstm_step32_fwd_kernel"), names.count("lstm_step32_bwd_kernel")) == (T if one else 0, T)
