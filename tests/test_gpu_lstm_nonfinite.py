"""GPU: an infinity or a NaN in one sample of a batch stays in that sample, in every form of the bf16 recurrences: the
other samples' h, c, gates and dx are those of the clean batch, bit for bit (a sample's sums take no term of another, and
their order does not depend on values)."""
import numpy as np
import pytest
import torch

from paper_2203_05705_amd import binding as ard
from util import from_vals, stored

pytestmark = pytest.mark.gpu

# a batch block per XCD: 16 and 24 units per workgroup, 8 and 16 rows, whole and partly filled shares of the last wavefronts
# (25, 31 and 22 workgroups; 23 with padding units); staging wavefronts; without them; a launch per step
FORMS = [(4, 20, 600, {}), (4, 128, 600, {}), (4, 20, 744, {}), (4, 100, 528, {}), (4, 60, 545, {}), (4, 20, 768, {}), (4, 20, 300, {}), (4, 128, 300, {}),
         (4, 128, 520, {"ARD_LSTM_SPREAD": "1"}), (4, 200, 200, {}), (3, 20, 1020, {}), (3, 16, 1100, {}), (3, 256, 512, {}), (3, 20, 600, {"ARD_NO_PERSIST": "1"})]


def _layer(T, B, H):
    rng = np.random.default_rng(T + B + H)
    I = 24
    x, dh = (from_vals(stored(rng.standard_normal(s), "bf16"), "bf16") for s in ((T, B, I), (T, B, H)))
    return x, dh, from_vals(stored(rng.uniform(-0.06, 0.06, (4 * H, I + H)), "bf16"), "bf16"), ard.Pattern.row(1, 1)


@pytest.mark.parametrize("value", [float("inf"), float("nan")])
@pytest.mark.parametrize("T,B,H,env", FORMS)
def test_a_sample_that_is_not_finite_stays_alone(T, B, H, env, value, monkeypatch):
    for k, v in env.items():
        monkeypatch.setenv(k, v)
    x, dh, W, pat = _layer(T, B, H)
    h, c, g = ard.lstm_fwd(x, W, pat)
    dx, _ = ard.lstm_bwd(x, W, pat, h, c, g, dh)
    for row in sorted({0, 3, 7 % B, B - 1}):
        print("lstm, one sample not finite", T, B, H, env, value, "row", row, flush=True)
        others = [r for r in range(B) if r != row]
        bad_dh, bad_x = dh.clone(), x.clone()
        bad_dh[T - 1, row, : 40] = value   # units of the first workgroups
        got, _ = ard.lstm_bwd(x, W, pat, h, c, g, bad_dh)
        assert torch.equal(got[:, others], dx[:, others]), "dx of other samples"
        assert not torch.isfinite(got[0, row].float()).any(), "the sample's own dx"
        bad_x[0, row, 0] = value
        for a, b, what in zip(ard.lstm_fwd(bad_x, W, pat), (h, c, g), ("h", "c", "gates")):
            assert torch.equal(a[:, others], b[:, others]), what + " of other samples"
