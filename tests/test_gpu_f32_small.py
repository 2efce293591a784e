"""GPU parity of the fp32 products where their kernels branch: contractions of every number of 16-deep steps a wavefront of a
small tile takes at once or in rounds, outputs that own one to many positions, and large tiles that leave in runs of four
columns.  Every output starts poisoned; bounds are the fp32 ones of all products."""
import numpy as np
import pytest
import torch

from oracle import gemm as G
from oracle import patterns as P
from paper_2203_05705_amd import binding as ard
from test_gpu_gemm import _run_row_case
from util import assert_parity, from_vals, stored

pytestmark = pytest.mark.gpu

# Kept contraction indices: below a step, one step, 64 to a step of each of the four wavefronts, remainders, 4 and 8 steps
# each (what the two small tiles hold), 6 and 14 (what they take in two goes), and more.
KEPT = [1, 15, 16, 17, 63, 64, 65, 127, 256, 257, 383, 384, 385, 448, 449, 511, 512, 513, 575, 640, 831, 895, 896, 897, 960, 1100]


@pytest.mark.parametrize("step", [2, 3])
@pytest.mark.parametrize("kept", KEPT)
def test_contractions_of_few_steps(kept, step):
    # the last kept index is the operand's last one (b = step fills the last group, b = 1 ends with a group of one)
    n, pat = (kept * step, (step, step)) if kept == 1 or kept % 2 == 0 else ((kept - 1) * step + 1, (step, 1))
    _run_row_case("f32", 19, n, 37, (2, 2), pat, alpha=1.25, seed=kept)         # forward
    _run_row_case("f32", 18, 70, n, pat, (3, 1), alpha=-0.5, seed=kept)         # data gradient
    _run_row_case("f32", kept, 45, 75, (2, 1), (step, step), seed=kept)         # weight gradient


@pytest.mark.parametrize("po,pi", [(None, None), ((2, 1), None), (None, (4, 3)), ((2, 2), (2, 1)), ((4, 4), None), ((3, 1), (2, 2)), ((8, 5), None)])
@pytest.mark.parametrize("B,I,O", [(1, 9, 17), (16, 32, 16), (17, 63, 31), (40, 65, 130)])
def test_small_outputs_store_the_zeros_they_own(B, I, O, po, pi):
    _run_row_case("f32", B, I, O, po, pi, alpha=1.5, relu=True, seed=B, use_relu_src=True)


@pytest.mark.parametrize("po,pi", [(None, None), ((2, 1), (2, 2)), ((3, 3), None), (None, (5, 2)), ((8, 3), (2, 1))])
@pytest.mark.parametrize("B,I,O", [(70, 1027, 1030), (516, 771, 1153)])
def test_large_outputs_leave_in_runs(B, I, O, po, pi):
    _run_row_case("f32", B, I, O, po, pi, alpha=-0.75, relu=True, seed=O, use_relu_src=True)


@pytest.mark.parametrize("I", [1030, 1027])
def test_large_outputs_with_listed_rows(I):
    B, O = 66, 1100
    rng = np.random.default_rng(I)
    keep = np.sort(rng.choice(O, 531, replace=False)).astype(np.int32)
    mo, mi = np.zeros(O, np.uint8), P.row_mask(I, 2, 1)
    mo[keep] = 1
    X, dY = (stored(rng.standard_normal(s), "f32") for s in ((B, I), (B, O)))
    dW = torch.full((O, I), float("nan"), device="cuda")
    ard.drop_gemm_bwd_weight(from_vals(dY, "f32"), from_vals(X, "f32"), ard.Pattern.list(torch.from_numpy(keep).cuda()), ard.Pattern.row(2, 1), out=dW)
    MW = G.weight_mask_rows(mo, mi)
    assert_parity(dW, G.drop_gemm_bwd_weight(dY, X, MW, mo), "f32", zero_mask=MW == 0, what="dW")
