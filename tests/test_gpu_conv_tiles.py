"""GPU parity of the bf16 convolutions in every tile shape their launch chooses from (by rows and output pixels) and in every
way a tile leaves: planes of whole 16-byte pieces, of whole words, of an odd number of pixels, and an output at an odd place."""
import numpy as np
import pytest
import torch

from oracle import conv as OC
from paper_2203_05705_amd import binding as ard
from util import assert_parity, from_vals, stored

pytestmark = pytest.mark.gpu

# pixels 28 x 28 = 49 pieces, 14 x 14 = 49 half pieces, 13 x 13 odd; channels on the wide side; tile of the wide side's product
CASES = [(3, 28, 90), (2, 13, 140), (76, 28, 100), (76, 14, 129), (100, 28, 101), (450, 13, 97), (128, 28, 65), (540, 14, 127), (590, 13, 80),
         (40, 28, 200), (160, 14, 131), (60, 28, 256), (280, 13, 133), (80, 28, 250), (330, 14, 140), (400, 13, 135)]


@pytest.mark.parametrize("N,S,wide", CASES)
def test_every_tile_shape(N, S, wide):
    print("conv tiles", N, S, wide, flush=True)
    rng = np.random.default_rng(N + wide)
    narrow, k, pad = 12, 1 if N * S * S > 20000 else 3, 0 if N * S * S > 20000 else 1
    for C, Cout in ((narrow, wide), (wide, narrow)):  # wide: rows of the forward product, then of the data gradient
        A, Wt, dY = (stored(rng.standard_normal(s) * 0.5, "bf16") for s in ((N, C, S, S), (Cout, C, k, k), (N, Cout, S, S)))
        m = np.ones(C, np.uint8)
        m[rng.choice(C, C // 8, replace=False)] = 0
        keep, cnt = torch.from_numpy(np.flatnonzero(m).astype(np.int32)).cuda(), int(m.sum())
        Ad, Wd, dYd = (from_vals(v, "bf16") for v in (A, Wt, dY))
        if C == narrow:
            out = torch.full((N, Cout, S, S), float("nan"), dtype=torch.bfloat16, device="cuda")
            assert_parity(ard.conv_fwd(Ad, Wd, keep, cnt, 1, pad, out=out), OC.conv_fwd(A, Wt, m, 1, pad), "bf16", None, "Y")
        else:
            assert_parity(ard.conv_bwd_data(dYd, Wd, keep, cnt, (S, S), 1, pad), OC.conv_bwd_data(dY, Wt, m, (S, S), 1, pad), "bf16",
                          np.broadcast_to((m == 0)[None, :, None, None], A.shape), "dA")


@pytest.mark.parametrize("S", [8, 14, 13])
def test_output_at_an_odd_place(S):
    rng = np.random.default_rng(S)
    N, C, Cout = 5, 20, 150
    A, Wt = stored(rng.standard_normal((N, C, S, S)) * 0.5, "bf16"), stored(rng.standard_normal((Cout, C, 3, 3)) * 0.5, "bf16")
    m = np.ones(C, np.uint8)
    flat = torch.full((N * Cout * S * S + 2,), float("nan"), dtype=torch.bfloat16, device="cuda")
    out = flat[1:-1].view(N, Cout, S, S)
    ard.conv_fwd(from_vals(A, "bf16"), from_vals(Wt, "bf16"), torch.arange(C, dtype=torch.int32, device="cuda"), C, 1, 1, out=out)
    assert_parity(out, OC.conv_fwd(A, Wt, m, 1, 1), "bf16", None, "Y")
    assert torch.isnan(flat[0]) and torch.isnan(flat[-1])


# listed pixels: scattered ones (2 bytes at a time) and bands (pieces, pairs across a band's end, odd bands) in wide and narrow tiles
@pytest.mark.parametrize("N,C,Cout,H,W,x,p", [(3, 64, 100, 14, 14, 14, 0.4), (2, 64, 140, 13, 13, 26, 0.5), (40, 64, 150, 16, 16, 16, 0.9), (30, 64, 80, 28, 28, 84, 0.7),
                                              (12, 64, 256, 28, 28, 28, 0.5)])
def test_listed_pixels(N, C, Cout, H, W, x, p):
    from oracle import sensitivity as SE
    rng = np.random.default_rng(H + Cout)
    A, Wt = stored(rng.standard_normal((N, C, H, W)) * 0.5, "bf16"), stored(rng.standard_normal((Cout, C, 3, 3)) * 0.5, "bf16")
    Ad, Wd = from_vals(A, "bf16"), from_vals(Wt, "bf16")
    mask = (rng.uniform(size=(N, H * W)) < p).astype(np.uint8)
    keep = torch.from_numpy(np.flatnonzero(mask).astype(np.int32)).cuda()
    Y = ard.conv_fwd_rows(Ad, Wd, dict(mask=torch.from_numpy(mask.reshape(-1)).cuda(), keep=keep), int(mask.sum()), 1, 1)
    assert_parity(Y, SE.conv_fwd_rows(A, Wt, mask, 1, 1), "bf16", None, "Y rows")
    _, RB, CB = ard.sens_regions(A.shape, (3, 3), 1, 1, x, 64 * 9)
    blk = (rng.uniform(size=(N, RB, CB)) < p).astype(np.uint8)
    Y = ard.conv_fwd_blocks(Ad, Wd, torch.from_numpy(blk.reshape(-1)).cuda(), x, 64 * 9, 1, 1)
    assert_parity(Y, SE.conv_fwd_blocks(A, Wt, blk, x, 64 * 9, 1, 1), "bf16", None, "Y blocks")
