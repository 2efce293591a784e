"""GPU parity of fp32 products in tiles of 32 x 32 whose results lie among dropped columns and leave in runs of four: strided and compact
operands, runs cut at the rows' ends, dropped rows, the ReLU mask of a gradient."""
import numpy as np
import pytest
import torch

from paper_2203_05705_amd import binding as ard
from test_gpu_gemm import _run_row_case
from util import assert_parity

pytestmark = pytest.mark.gpu

PATTERNS = [((3, 3), (3, 1)), ((2, 1), (2, 2)), ((5, 2), (5, 5)), ((1, 1), (4, 3))]


@pytest.mark.parametrize("po,pi", PATTERNS)
@pytest.mark.parametrize("B,I,O", [(128, 1030, 1027), (33, 517, 770)])
def test_strided_operands(B, I, O, po, pi):
    _run_row_case("f32", B, I, O, po, pi, alpha=0.75, relu=True, seed=B + I, use_relu_src=True)


@pytest.mark.parametrize("po,pi", PATTERNS)
@pytest.mark.parametrize("B,I,O", [(128, 2048, 2048), (130, 1501, 1203), (30, 1024, 3000)])
def test_weight_gradient_of_compact_operands(B, I, O, po, pi):
    g = torch.Generator(device="cuda").manual_seed(B + I)
    rows, cols = torch.arange(po[1] - 1, O, po[0], device="cuda"), torch.arange(pi[1] - 1, I, pi[0], device="cuda")
    dY, X = (torch.randn((B, len(k)), generator=g, device="cuda") for k in (rows, cols))
    dW = torch.full((O, I), float("nan"), device="cuda")
    ard.drop_gemm_bwd_weight(ard.pad_compact(dY), ard.pad_compact(X), ard.Pattern.row(*po), ard.Pattern.row(*pi), flags=ard.IN_COMPACT | ard.OUT_COMPACT,
                             I=I, O=O, out=dW)
    ref = torch.zeros((O, I), dtype=torch.float64, device="cuda")
    ref[rows[:, None], cols[None, :]] = dY.double().t() @ X.double()
    assert_parity(dW, ref.cpu().numpy(), "f32", zero_mask=(ref == 0).cpu().numpy(), what="dW")
