"""GPU parity of the bf16 recurrences with a batch block per XCD at the edges of their range: blocks of 8 and 16 rows, one
row and ragged last blocks, 16 and 24 units per workgroup, every number of slices per wavefront, an odd number of
workgroups, padding units; and with device-scope stores, as if the workgroups of a block were on several XCDs."""
import numpy as np
import pytest

from oracle import patterns as P
from paper_2203_05705_amd import binding as ard
from test_gpu_lstm import _check
from util import from_vals, stored

pytestmark = pytest.mark.gpu

SHAPES = [(4, 1, 8, 1), (3, 8, 130, 1), (3, 9, 264, 2), (3, 64, 257, 1), (3, 65, 257, 1), (3, 33, 504, 3), (3, 127, 512, 1), (3, 64, 513, 1),
          (3, 7, 529, 1), (3, 65, 536, 1), (3, 90, 600, 1), (4, 128, 600, 1), (3, 24, 768, 1), (3, 80, 768, 1), (4, 128, 1024, 2)]


def _layer(T, B, H, dp):
    print("lstm, a block per XCD", T, B, H, dp, flush=True)
    rng = np.random.default_rng(T + B + H)
    I = 24
    x, dh = (stored(rng.standard_normal(s), "bf16") for s in ((T, B, I), (T, B, H)))
    W = stored(rng.uniform(-0.06, 0.06, (4 * H, I + H)), "bf16")
    _check("bf16", x, W, dh, P.row_mask(H, dp, dp), ard.Pattern.row(dp, dp), *(from_vals(v, "bf16") for v in (x, W, dh)), f"xcd {B} {H}")


@pytest.mark.parametrize("T,B,H,dp", SHAPES)
def test_recurrences_with_a_block_per_xcd(T, B, H, dp):
    _layer(T, B, H, dp)


@pytest.mark.parametrize("T,B,H,dp", [(3, 40, 520, 1), (3, 128, 512, 2)])
def test_recurrences_of_a_spread_block(T, B, H, dp, monkeypatch):
    monkeypatch.setenv("ARD_LSTM_SPREAD", "1")
    _layer(T, B, H, dp)
