"""GPU parity of the bf16 products where a tile leaves in different ways: whole 16-byte pieces, rows that begin at odd places,
the last columns of ragged widths, the ReLU mask of a gradient, an output that is added to, partial sums, kept columns spread
among zeros, and tiles of a tile pattern; in the smallest and the largest tiles.  Outputs start poisoned."""
import numpy as np
import pytest
import torch

from oracle import gemm as G
from oracle import patterns as P
from paper_2203_05705_amd import binding as ard
from test_gpu_gemm import _run_row_case
from util import assert_parity, from_vals, stored

pytestmark = pytest.mark.gpu

SIZES = [(64, 64, 64), (65, 72, 130), (70, 135, 67), (16, 1472, 368), (257, 194, 321), (300, 513, 1030), (1030, 1028, 772), (2048, 2050, 2047)]


@pytest.mark.parametrize("B,I,O", SIZES)
def test_plain(B, I, O):
    _run_row_case("bf16", B, I, O, None, None, alpha=-1.25, relu=True, seed=B, use_relu_src=True)


@pytest.mark.parametrize("B,I,O", SIZES[:-1])
def test_added_to(B, I, O):
    _run_row_case("bf16", B, I, O, None, None, alpha=0.5, beta=-0.75, seed=O, use_relu_src=True)


@pytest.mark.parametrize("po,pi", [((2, 1), None), (None, (3, 2)), ((3, 3), (2, 2)), ((8, 5), (8, 8)), ((9, 4), None)])
@pytest.mark.parametrize("B,I,O", [(40, 90, 75), (130, 515, 263), (1027, 1030, 600)])
def test_spread_among_zeros(B, I, O, po, pi):
    _run_row_case("bf16", B, I, O, po, pi, alpha=1.5, relu=True, seed=I, use_relu_src=True)


@pytest.mark.parametrize("B,I,O,t,dp,b", [(66, 192, 256, 32, 2, 1), (70, 320, 192, 64, 3, 2), (200, 200, 136, 32, 4, 3), (1024, 2048, 1024, 64, 2, 2)])
def test_tiles(B, I, O, t, dp, b):
    rng = np.random.default_rng(O)
    X, W, dY, src = (stored(rng.standard_normal(s) * 0.5, "bf16") for s in ((B, I), (O, I), (B, O), (B, I)))
    MW = P.expand_tile_mask(P.tile_mask(O, I, t, t, dp, b), O, I, t, t).astype(np.float64)
    pat = ard.Pattern.tile(dp, b, t, t)
    ones = np.ones(O, np.uint8)
    Xd, Wd, dYd, sd = (from_vals(v, "bf16") for v in (X, W, dY, src))
    new = lambda *s: torch.full(s, float("nan"), dtype=torch.bfloat16, device="cuda")
    assert_parity(ard.drop_gemm_fwd(Xd, Wd, pat, relu=True, out=new(B, O)), G.drop_gemm_fwd(X, W, MW, ones, 1.0, True), "bf16", what="Y")
    assert_parity(ard.drop_gemm_bwd_data(dYd, Wd, pat, relu_src=sd, out=new(B, I)), G.relu_bwd(G.drop_gemm_bwd_data(dY, W, MW, ones), src), "bf16", what="dX")
    assert_parity(ard.drop_gemm_bwd_weight(dYd, Xd, pat, out=new(O, I)), G.drop_gemm_bwd_weight(dY, X, MW, ones), "bf16", zero_mask=MW == 0, what="dW")
