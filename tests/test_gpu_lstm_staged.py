"""GPU parity of the bf16 recurrences with staging wavefronts at the edges of their range (batches above 128, more than
768 kept units, or two steps forward of more than 512): 8 and 16 units per workgroup, every number of slices per wavefront, slices that end inside a share and
ragged batch blocks; and beyond it (1025 units and more, too many workgroups), where the recurrences without staging
wavefronts run."""
import numpy as np
import pytest

from oracle import lstm as L
from oracle import patterns as P
from oracle import rounding as R
from paper_2203_05705_amd import binding as ard
from test_gpu_lstm import _check
from util import CEILING, assert_parity, from_vals, max_rel_err, stored, to_host

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T,B,H,dp", [(4, 1, 8, 1), (3, 17, 129, 1), (4, 40, 260, 1), (3, 33, 513, 1), (3, 20, 760, 1), (3, 33, 1020, 1), (3, 128, 600, 1),
                                      (3, 128, 1024, 1), (3, 16, 1100, 1), (4, 100, 1030, 2)])
def test_staged_recurrences(T, B, H, dp):
    """Both ends of the recurrences' ranges; those of up to 768 kept units and 128 rows run with a batch block per XCD."""
    print("staged lstm", T, B, H, dp, flush=True)
    rng = np.random.default_rng(T + B + H)
    I = 16
    x, dh = (stored(rng.standard_normal(s), "bf16") for s in ((T, B, I), (T, B, H)))
    W = stored(rng.uniform(-0.06, 0.06, (4 * H, I + H)), "bf16")
    _check("bf16", x, W, dh, P.row_mask(H, dp, 1), ard.Pattern.row(dp, 1), *(from_vals(v, "bf16") for v in (x, W, dh)), f"staged {B} {H}")


# (T, B, H) and the slices per wavefront of the kernels with staging wavefronts, forward (units per workgroup / 8, slices)
# and backward, None where another form takes the pass
STAGED = [((3, 200, 128), (1, 4), 4), ((3, 200, 200), (1, 4), 8), ((4, 160, 400), (1, 8), 16), ((3, 300, 256), (2, 4), None), ((3, 160, 500), (2, 8), None),
          ((3, 160, 760), (2, 12), None), ((3, 129, 405), (1, 8), 16), ((3, 128, 1000), (2, 16), None), ((3, 50, 800), (1, 16), 32),
          ((2, 20, 600), (1, 12), None), ((2, 96, 513), (1, 12), None), ((2, 65, 768), (2, 12), None)]


@pytest.mark.parametrize("shape", [s for s, _, _ in STAGED])
def test_staged_recurrences_of_every_length(shape):
    T, B, H = shape
    print("staged lstm, every length", shape, flush=True)
    rng = np.random.default_rng(T + B + H)
    I = 16
    x, dh = (stored(rng.standard_normal(s), "bf16") for s in ((T, B, I), (T, B, H)))
    W = stored(rng.uniform(-0.06, 0.06, (4 * H, I + H)), "bf16")
    _check("bf16", x, W, dh, P.row_mask(H, 1, 1), ard.Pattern.row(1, 1), *(from_vals(v, "bf16") for v in (x, W, dh)), f"staged {B} {H}")


# (T, B, H): forward, backward without staging wavefronts.  Forward: 32, 64 and 128 batch rows per workgroup, the state read
# with device-scope loads and through L2; backward: 16, 32 and 64 rows, the same two ways.
BEYOND_FWD = [(3, 16, 1100), (3, 32, 1400), (3, 33, 1030), (3, 64, 1030), (3, 640, 200), (3, 192, 680), (3, 2048, 128), (3, 1024, 256),
              (3, 1160, 200)]
BEYOND_BWD = [(3, 16, 1100), (3, 48, 1100), (3, 256, 512), (3, 116, 576), (3, 128, 600), (3, 2048, 128), (3, 1160, 200), (3, 2048, 256), (3, 2080, 128)]


@pytest.mark.parametrize("T,B,H", sorted(set(BEYOND_FWD + BEYOND_BWD)))
def test_recurrences_without_staging_wavefronts(T, B, H):
    """Tolerances of _check, but for single elements of dW a bound of their own: dW is a sum of T * B products of a gate
    gradient and an input, both stored in bf16, and where fp32 sums in another order fall on the other side of a rounding
    boundary each is off by one unit in the last place, 2^-7 of its size.  So |d| <= 2^-6 sum |dgate||input| + 2^-8 |dW|;
    of the million elements of the widest layers some are what is left of terms that cancel (2.3e-2 of the rms where
    CEILING allows 2e-2), and the sum of the terms' sizes says by how much."""
    print("lstm beyond the staged recurrences", T, B, H, flush=True)
    rng = np.random.default_rng(B + H)
    I = 16
    x, dh = (stored(rng.standard_normal(s), "bf16") for s in ((T, B, I), (T, B, H)))
    W = stored(rng.uniform(-0.06, 0.06, (4 * H, I + H)), "bf16")
    xd, Wd, dhd = (from_vals(v, "bf16") for v in (x, W, dh))
    m, pat = P.row_mask(H, 1, 1), ard.Pattern.row(1, 1)
    fwd = L.lstm_forward(x, W, m, R.to_bf16_values)
    dgates = []   # as the oracle stores them, last step first

    def store(a):
        dgates.append(R.to_bf16_values(a))
        return dgates[-1]
    bwd = L.lstm_backward(x, W, m, fwd, dh, store)
    h, c, gates = ard.lstm_fwd(xd, Wd, pat)
    dx, dW = ard.lstm_bwd(xd, Wd, pat, h, c, gates, dhd)
    lim = dict(tol=CEILING["bf16"], etol=CEILING["bf16"])
    for got, ref, what in ((h, fwd["h"], "h"), (c, fwd["c"], "c"), (gates, fwd["gates"], "gates"), (dx, bwd["dx"], "dx")):
        assert_parity(got, ref, "bf16", None, f"beyond {B} {H} {what}", **lim)
    sizes = np.zeros_like(bwd["dW"])
    for t, d in zip(range(T - 1, -1, -1), dgates):
        sizes += np.abs(d).T @ np.abs(np.concatenate([x[t], fwd["h"][t - 1] if t > 0 else np.zeros((B, H))], axis=1))
    got = to_host(dW)
    assert np.all(np.isfinite(got)) and max_rel_err(got, bwd["dW"]) <= CEILING["bf16"]
    worst = np.max(np.abs(got - bwd["dW"]) - 2.0 ** -6 * sizes - 2.0 ** -8 * np.abs(bwd["dW"]))
    assert worst <= 1e-6 * np.max(sizes), (B, H, worst)   # (fp32 sums of the terms themselves)
