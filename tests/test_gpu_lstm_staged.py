"""GPU parity of the bf16 recurrences with staging wavefronts at the edges of their range: 8 and 16 units per workgroup,
every number of slices per wavefront, slices that end inside a share, one batch row and ragged batch blocks; and just
beyond it (1025 units and more, too many workgroups), where the recurrences without staging wavefronts run."""
import numpy as np
import pytest

from oracle import patterns as P
from paper_2203_05705_amd import binding as ard
from test_gpu_lstm import _check
from util import from_vals, stored

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T,B,H,dp", [(4, 1, 8, 1), (3, 17, 129, 1), (4, 40, 260, 1), (3, 33, 513, 1), (3, 20, 760, 1), (3, 33, 1020, 1), (3, 128, 600, 1),
                                      (3, 128, 1024, 1), (3, 16, 1100, 1), (4, 100, 1030, 2)])
def test_staged_recurrences(T, B, H, dp):
    print("staged lstm", T, B, H, dp, flush=True)
    rng = np.random.default_rng(T + B + H)
    I = 16
    x, dh = (stored(rng.standard_normal(s), "bf16") for s in ((T, B, I), (T, B, H)))
    W = stored(rng.uniform(-0.06, 0.06, (4 * H, I + H)), "bf16")
    _check("bf16", x, W, dh, P.row_mask(H, dp, 1), ard.Pattern.row(dp, 1), *(from_vals(v, "bf16") for v in (x, W, dh)), f"staged {B} {H}")
