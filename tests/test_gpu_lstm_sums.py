"""GPU parity of LSTM weight gradients added from partial sums, the number of them asserted case by case: one, odd ones and whole groups,
units next to each other and apart from either parity, rows that end in the middle of a 16-byte piece, dropped tiles."""
import numpy as np
import pytest

import dryrun as D
from paper_2203_05705_amd import binding as ard
from test_gpu_lstm import _check_tile
from test_gpu_lstm_spread import _case
from util import stored

pytestmark = pytest.mark.gpu


def _sums(T, B, I, H, dp, b, tile):
    with D.dry_run() as lib:
        p = D.FakeHeap()(1 << 20)
        _, r = D.cpat((dp, b), ard.PAT_TILE, (tile, tile)) if tile else D.cpat((dp, b))
        n = lib.ard_lstm_workspace_bytes(D.BF16, T, B, I, H, r)
        D.launches(lib)
        assert lib.ard_lstm_bwd(D.BF16, T, B, I, H, p, p, r, p, p, p, p, p, p, p, n, None) == 0
        return [i for i in D.instances(lib) if i.startswith("lstm_scatter_dw_kernel")]


@pytest.mark.parametrize("T,B,I,H,dp,b,x,h", [
    (24, 160, 1200, 1200, 1, 1, 1, 1), (24, 160, 700, 1200, 1, 1, 2, 1), (32, 128, 801, 801, 1, 1, 2, 2), (32, 128, 998, 1400, 2, 1, 2, 3), (24, 192, 804, 700, 1, 1, 3, 3),
    (32, 192, 900, 1600, 3, 2, 3, 4), (48, 160, 801, 1000, 2, 2, 4, 6), (32, 192, 900, 1000, 2, 1, 4, 7), (64, 128, 1200, 1400, 4, 3, 4, 8)])
def test_units(T, B, I, H, dp, b, x, h):
    assert _sums(T, B, I, H, dp, b, 0) == [f"lstm_scatter_dw_kernel<{x}, {h}, 0>"]
    _case("bf16", T, B, I, H, dp, b, 0.03)


@pytest.mark.parametrize("T,B,I,H,dp,b,x,h", [(32, 128, 801, 801, 2, 2, 2, 2), (32, 128, 1000, 704, 3, 1, 2, 3)])
def test_dropped_tiles(T, B, I, H, dp, b, x, h):
    assert _sums(T, B, I, H, dp, b, 32) == [f"lstm_scatter_dw_kernel<{x}, {h}, 0>"]
    rng = np.random.default_rng(H)
    a, dh = (stored(rng.standard_normal((T, B, n)), "bf16") for n in (I, H))
    W = stored(rng.uniform(-0.03, 0.03, (4 * H, I + H)), "bf16")
    _check_tile("bf16", a, W, dh, (32, 32, dp, b), f"lstm tiles T={T} B={B} I={I} H={H} dp={dp}")
