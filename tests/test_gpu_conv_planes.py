"""GPU parity of the fp32 convolutions on zero-bordered channel planes, at the sizes where their kernels change
branch: channels around the 16-deep contraction steps, output rows that are and are not whole groups of four,
filters that keep, shrink and grow the image, one pixel and several tiles of pixels, split weight gradients, and
dY masked by the band-based patterns while it is copied."""
import numpy as np
import pytest
import torch

from oracle import conv as OC
from paper_2203_05705_amd import binding as ard
from util import assert_parity, from_vals, stored

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,C,Cout,H,W,k,pad,rate", [
    (1, 1, 1, 1, 1, 1, 0, 0.0), (1, 3, 2, 3, 3, 3, 0, 0.0), (2, 16, 16, 4, 4, 3, 1, 0.0), (3, 33, 17, 5, 8, 3, 2, 0.4),
    (2, 34, 65, 13, 11, 5, 2, 0.5), (9, 130, 129, 12, 16, 3, 1, 0.1), (40, 20, 18, 9, 7, 3, 1, 0.5), (1, 70, 260, 7, 7, 1, 0, 0.3),
    (16, 48, 130, 30, 30, 3, 1, 0.5)])
def test_planes(N, C, Cout, H, W, k, pad, rate):
    print("planes", N, C, Cout, H, W, k, pad, rate, flush=True)
    rng = np.random.default_rng(C * 100 + Cout)
    Ho, Wo = H + 2 * pad - k + 1, W + 2 * pad - k + 1
    A, Wt, dY = (stored(rng.standard_normal(s) * 0.5, "f32") for s in ((N, C, H, W), (Cout, C, k, k), (N, Cout, Ho, Wo)))
    A = np.maximum(A, 0)
    Ad, Wd, dYd = (from_vals(v, "f32") for v in (A, Wt, dY))
    sel = ard.conv_select(Ad, rate)
    m, cnt = sel["mask"].cpu().numpy(), int(sel["count"].item())
    ws = torch.full((ard.conv_workspace_bytes(ard.F32, N, C, H, W, Cout, k, k, 1, pad),), 0xFF, dtype=torch.uint8, device="cuda")
    assert_parity(ard.conv_fwd(Ad, Wd, sel["keep"], cnt, 1, pad, ws=ws), OC.conv_fwd(A, Wt, m, 1, pad), "f32", None, "Y")
    assert_parity(ard.conv_bwd_data(dYd, Wd, sel["keep"], cnt, (H, W), 1, pad, ws=ws), OC.conv_bwd_data(dY, Wt, m, (H, W), 1, pad), "f32",
                  np.broadcast_to((m == 0)[None, :, None, None], A.shape), "dA")
    assert_parity(ard.conv_bwd_weight(dYd, Ad, sel["keep"], cnt, (k, k), 1, pad, ws=ws), OC.conv_bwd_weight(dY, A, m, (k, k), 1, pad), "f32",
                  np.broadcast_to((m == 0)[None, :, None, None], Wt.shape), "dWt")
