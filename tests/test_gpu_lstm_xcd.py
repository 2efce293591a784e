"""GPU parity of the bf16 recurrences with a batch block per XCD at the edges of their range: blocks of 8 and 16 rows, one
row and ragged last blocks, 16 and 24 units per workgroup, every number of slices per wavefront, an odd number of
workgroups, padding units; with device-scope stores, as if the workgroups of a block were on several XCDs; with workgroups
that are not there; and on two streams at once."""
import numpy as np
import pytest
import torch

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


def _pass(T, B, H, seed):
    """A layer's inputs, and a function that runs both directions of it in a workspace of its own and returns the results."""
    rng = np.random.default_rng(seed)
    I, pat = 24, ard.Pattern.row(1, 1)
    x, dh = (from_vals(stored(rng.standard_normal(s), "bf16"), "bf16") for s in ((T, B, I), (T, B, H)))
    W = from_vals(stored(rng.uniform(-0.06, 0.06, (4 * H, I + H)), "bf16"), "bf16")
    ws = torch.empty(ard.lstm_workspace_bytes(ard.BF16, T, B, I, H, pat), dtype=torch.uint8, device="cuda")
    off = ard.lstm_status_offset(ard.BF16, T, B, I, H, pat)

    def run():
        h, c, g = ard.lstm_fwd(x, W, pat, ws=ws)
        status = [ws[off:off + 4].view(torch.int32).clone()]
        dx, dW = ard.lstm_bwd(x, W, pat, h, c, g, dh, ws=ws)
        status.append(ws[off:off + 4].view(torch.int32).clone())
        return (h, c, g, dx, dW), status
    return run


def _same(got, want, what):
    assert all(int(s.item()) == 0 for s in got[1]), f"{what}: a recurrence gave up"
    for a, b, name in zip(got[0], want[0], ("h", "c", "gates", "dx", "dW")):
        assert torch.equal(a, b), f"{what}: {name} differs in {int((a != b).sum())} entries"


@pytest.mark.parametrize("T,B,H,there", [(5, 20, 250, (1, 2, 9)), (5, 100, 250, (1, 9)), (5, 20, 500, (1, 17, 31)), (5, 128, 500, (3, 31)), (5, 20, 750, (1, 17, 31)),
                                         (5, 128, 760, (3, 31)), (5, 70, 600, (24,))])
def test_seats_of_absent_workgroups_are_taken(T, B, H, there, monkeypatch):
    """Only the first workgroups of every block run, as if others held the CUs: they do the whole recurrence, with the same
    results bit for bit (the same sums in the same order) and without giving up."""
    run = _pass(T, B, H, T + B + H)
    want = run()
    for n in there:
        print("lstm, absent workgroups", T, B, H, n, flush=True)
        monkeypatch.setenv("ARD_LSTM_SEATS", str(n))
        _same(run(), want, f"{B} x {H}, {n} workgroups of a block")


def test_recurrences_on_two_streams_at_once():
    """Layers that each want all CUs of some XCDs, or of all of them, passing each other on two streams."""
    layers = [_pass(*s, seed=i) for i, s in enumerate([(20, 20, 750), (20, 20, 750), (12, 128, 512), (12, 60, 600)])]
    want = [run() for run in layers]
    torch.cuda.synchronize()
    streams = [torch.cuda.Stream() for _ in range(2)]
    print("recurrences on two streams", flush=True)
    got = []
    for _ in range(4):
        for first, second in ((0, 1), (2, 3), (0, 2), (1, 3)):
            for stream, k in zip(streams, (first, second)):
                with torch.cuda.stream(stream):
                    got.append((k, layers[k]()))
        torch.cuda.synchronize()
    for k, results in got:
        _same(results, want[k], f"layer {k}")
