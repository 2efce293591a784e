"""GPU parity: channel selection at the edges of its one-workgroup search (wavefronts, 1024 maps, the LDS staging) and with
scores that agree in their leading bits or altogether."""
import numpy as np
import pytest

from oracle import conv as OC
from paper_2203_05705_amd import binding as ard
from util import from_vals, stored

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("values", ["spread", "all equal", "few values", "many zeros", "low bits", "largest"])
@pytest.mark.parametrize("C", [1, 5, 64, 65, 389, 1024, 1025, 4096, 4097])
def test_select(C, values):
    print(f"select C={C} {values}", flush=True)
    rng = np.random.default_rng(C)
    A = {"spread": lambda: rng.standard_normal((2, C, 3, 3)),
         "all equal": lambda: np.full((2, C, 3, 3), 0.5),
         "few values": lambda: np.repeat(rng.integers(1, 4, C), 18).reshape(C, 2, 3, 3).swapaxes(0, 1),
         "many zeros": lambda: rng.standard_normal((2, C, 3, 3)) * (rng.random((1, C, 1, 1)) < 0.4),
         "low bits": lambda: np.where(np.arange(18).reshape(2, 1, 3, 3) > 0, 32768.0, rng.integers(0, 7, (1, C, 1, 1)) * 2.0 ** -24),
         "largest": lambda: np.where(rng.random((1, C, 1, 1)) < 0.5, np.inf, rng.standard_normal((2, C, 3, 3)) * 3e4)}[values]()
    Av = np.where(np.isinf(A), A, stored(np.where(np.isinf(A), 0, A), "f32"))
    Ad = from_vals(Av, "f32")
    for rate in (0.0, 1.0 / max(C, 2), 0.3, 0.5, 0.7, 1.0):
        sel = ard.conv_select(Ad, rate)
        score = OC.channel_score_fixed(Av)
        m = OC.select_channels(score, rate)
        keep = np.flatnonzero(m)
        assert np.array_equal(sel["score"].cpu().numpy(), score)
        assert np.array_equal(sel["mask"].cpu().numpy(), m)
        assert int(sel["count"].item()) == len(keep)
        assert np.array_equal(sel["keep"].cpu().numpy()[:len(keep)], keep)
