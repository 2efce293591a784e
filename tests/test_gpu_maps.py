"""GPU parity of the products whose operands or outputs are not whole 16-byte rows, at the sizes where their
kernels change branch: fp32 tiles of every shape with partial rows, columns and contraction steps, strided and
listed maps; bf16 operands that are copied compact first; outputs whose rows have any length and alignment."""
import numpy as np
import pytest
import torch

from oracle import gemm as G
from oracle import patterns as P
from paper_2203_05705_amd import binding as ard
from util import assert_parity, from_vals, stored

pytestmark = pytest.mark.gpu

# B, I, O, dp_out, dp_in: one element, a contraction below one step, edges of 16 / 32 / 64 / 128 tiles, rows shorter
# than a group of four, a split contraction (many rows, few outputs), copies before the product, wide periods
SHAPES = [(1, 1, 1, 1, 1), (3, 5, 2, 1, 1), (16, 16, 16, 1, 1), (17, 33, 19, 2, 3), (64, 100, 130, 3, 1), (129, 257, 131, 1, 2),
          (260, 513, 777, 5, 4), (2050, 40, 24, 2, 1), (515, 1030, 1027, 2, 2), (1029, 770, 900, 1, 1), (70, 300, 290, 9, 8), (40, 97, 63, 8, 8)]


def _layer(dtype, B, I, O, po, pi, mo, mi, seed, relu_src):
    rng = np.random.default_rng(seed)
    X, W, dY, S = (stored(rng.standard_normal(s) * 0.5, dtype) for s in ((B, I), (O, I), (B, O), (B, I)))
    MW = G.weight_mask_rows(mo, mi)
    Xd, Wd, dYd, Sd = (from_vals(v, dtype) for v in (X, W, dY, S))
    assert_parity(ard.drop_gemm_fwd(Xd, Wd, po, pi, relu=True), G.drop_gemm_fwd(X, W, MW, mo, 1.0, relu=True), dtype,
                  zero_mask=(mo == 0)[None, :], what="Y")
    dX = G.drop_gemm_bwd_data(dY, W, MW, mo, 1.0)
    if relu_src:
        assert_parity(ard.drop_gemm_bwd_data(dYd, Wd, po, pi, relu_src=Sd), dX * (S > 0), dtype, zero_mask=(S <= 0) | (mi == 0)[None, :], what="dX")
    else:
        assert_parity(ard.drop_gemm_bwd_data(dYd, Wd, po, pi), dX, dtype, zero_mask=(mi == 0)[None, :], what="dX")
    assert_parity(ard.drop_gemm_bwd_weight(dYd, Xd, po, pi), G.drop_gemm_bwd_weight(dY, X, MW, mo), dtype, zero_mask=(MW == 0), what="dW")


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("shape", SHAPES, ids=str)
def test_row_patterns_on_any_size(shape, dtype):
    B, I, O, dp, dpi = shape
    dp, dpi = min(dp, O), min(dpi, I)
    b, bi = 1 + (I + O) % dp, 1 + (B + O) % dpi
    _layer(dtype, B, I, O, ard.Pattern.row(dp, b), ard.Pattern.row(dpi, bi), P.row_mask(O, dp, b), P.row_mask(I, dpi, bi), 7, B % 2 == 0)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_list_patterns_on_any_size(dtype):
    rng = np.random.default_rng(3)
    mo, mi = (rng.random(203) < 0.4).astype(np.uint8), (rng.random(149) < 0.5).astype(np.uint8)
    po, pi = (ard.Pattern.list(torch.from_numpy(P.keep_list(m)).cuda()) for m in (mo, mi))
    _layer(dtype, 65, 149, 203, po, pi, mo, mi, 4, False)


@pytest.mark.parametrize("B,I,O,x,y,dp,b", [(33, 96, 64, 32, 32, 2, 1), (130, 200, 333, 32, 32, 3, 2), (257, 417, 259, 64, 64, 5, 4),
                                            (64, 500, 290, 96, 160, 2, 2), (200, 700, 650, 128, 64, 7, 3), (20, 130, 1000, 256, 32, 4, 1)])
def test_fp32_tile_patterns(B, I, O, x, y, dp, b):
    """Tiles wider than the workgroup's tile, tile sizes that are no power of two, edge tiles of any width."""
    rng = np.random.default_rng(11)
    X, W, dY, S = (stored(rng.standard_normal(s) * 0.5, "f32") for s in ((B, I), (O, I), (B, O), (B, I)))
    MW = P.expand_tile_mask(P.tile_mask(O, I, x, y, dp, b), O, I, x, y).astype(np.float64)
    one = np.ones(O, np.uint8)
    pat = ard.Pattern.tile(dp, b, x, y)
    Xd, Wd, dYd, Sd = (from_vals(v, "f32") for v in (X, W, dY, S))
    assert_parity(ard.drop_gemm_fwd(Xd, Wd, pat, relu=True), G.drop_gemm_fwd(X, W, MW, one, 1.0, relu=True), "f32", what="Y")
    assert_parity(ard.drop_gemm_bwd_data(dYd, Wd, pat, relu_src=Sd), G.drop_gemm_bwd_data(dY, W, MW, one, 1.0) * (S > 0), "f32",
                  zero_mask=S <= 0, what="dX")
    assert_parity(ard.drop_gemm_bwd_weight(dYd, Xd, pat), G.drop_gemm_bwd_weight(dY, X, MW, one), "f32", zero_mask=(MW == 0), what="dW")
