"""fp32 convolutions with infinities and NaN among their inputs: they reach the sums that they are part of, and no
others (neighbouring rows, channels and images lie next to each other in the copies that the kernels read)."""
import numpy as np
import pytest
import torch
import torch.nn.functional as F

from paper_2203_05705_amd import binding as ard

pytestmark = pytest.mark.gpu


def _weight_gradient(dY, A, k, pad):
    """dW[co, c, r, s] in 64 bits: every output position against its own patch (zeros outside the image)."""
    N, Co = dY.shape[:2]
    cols = F.unfold(A.double(), k, padding=pad)                       # [N, C*k*k, positions]
    return torch.einsum("nol,ncl->oc", dY.double().reshape(N, Co, -1), cols).reshape(Co, A.shape[1], k, k)


def _same(got, want, what):
    got = got.double().cpu()
    for test in (torch.isnan, torch.isposinf, torch.isneginf):
        assert torch.equal(test(got), test(want)), f"{what}: {test.__name__} at {(test(got) != test(want)).nonzero()[:4].tolist()}"
    ok = torch.isfinite(want)
    scale = want[ok].abs().max()
    assert float((got[ok] - want[ok]).abs().max()) <= 1e-5 * float(scale), what


# filters that keep, shrink and grow the image; the corners and edges of the first and last plane; planes that end on a
# 16-position step and ones that do not; one channel more and one less than a group of 16
@pytest.mark.parametrize("N,C,Cout,H,W,k,pad", [(1, 8, 4, 8, 8, 3, 1), (2, 17, 16, 8, 8, 3, 0), (2, 15, 3, 7, 9, 3, 2), (3, 16, 33, 6, 6, 5, 2),
                                                (2, 3, 70, 14, 14, 1, 0), (1, 2, 2, 3, 1, 3, 2), (40, 20, 18, 9, 7, 3, 1)])
@pytest.mark.parametrize("value", [float("inf"), float("nan")])
def test_weight_gradient_keeps_them_where_they_belong(N, C, Cout, H, W, k, pad, value):
    print("nonfinite", N, C, Cout, H, W, k, pad, value, flush=True)
    g = torch.Generator().manual_seed(C * 10 + H)
    Ho, Wo = H + 2 * pad - k + 1, W + 2 * pad - k + 1
    A0, dY = torch.randn((N, C, H, W), generator=g), torch.randn((N, Cout, Ho, Wo), generator=g)
    keep = torch.arange(C, dtype=torch.int32, device="cuda")
    for at in {(0, min(5, C - 1), 0, 0), (0, 0, H - 1, W - 1), (N - 1, C - 1, H - 1, W - 1), (N - 1, C // 2, H // 2, 0), (N // 2, C - 1, 0, W - 1)}:
        A = A0.clone()
        A[at] = value
        got = ard.conv_bwd_weight(dY.cuda(), A.cuda(), keep, C, (k, k), 1, pad)
        _same(got, _weight_gradient(dY, A, k, pad), f"A{list(at)} = {value}")


def test_weight_gradient_over_kept_channels_and_bands():
    """The same through a kept list (a dropped channel's infinity is never read) and under a row pattern."""
    N, C, Co, H, W, k, pad = 3, 12, 5, 10, 7, 3, 1
    g = torch.Generator().manual_seed(3)
    A, dY = torch.randn((N, C, H, W), generator=g), torch.randn((N, Co, H, W), generator=g)
    A[1, 4, H - 1, W - 1] = float("inf")
    A[1, 7] = float("nan")
    kept = [0, 3, 4, 5, 9, 11]
    keep = torch.tensor(kept, dtype=torch.int32, device="cuda")
    want = torch.zeros((Co, C, k, k), dtype=torch.float64)
    want[:, kept] = _weight_gradient(dY, A[:, kept], k, pad)
    _same(ard.conv_bwd_weight(dY.cuda(), A.cuda(), keep, len(kept), (k, k), 1, pad), want, "kept channels")
