"""GPU parity of the bf16 products on large tiles at every number of contraction steps around the point from which their loads are
spread over the steps (whole and partial last steps), in all three operand layouts; and on the smallest tiles.
Reference: the same stored values multiplied in 64 bits."""
import numpy as np
import pytest
import torch

from paper_2203_05705_amd import binding as ard
from util import assert_parity

pytestmark = pytest.mark.gpu

STEPS = [64 * s for s in range(1, 12)] + [64 * 5 + 8, 64 * 7 + 40, 64 * 8 + 56]


def _random(g, *shape):
    return torch.randn(shape, generator=g, device="cuda").to(torch.bfloat16)


@pytest.mark.parametrize("M,N", [(2048, 3584), (3840, 3840), (1024, 1024)], ids=["256x128", "256x256", "64x64"])
@pytest.mark.parametrize("K", STEPS)
def test_dense_contraction_lengths(M, N, K):
    g = torch.Generator(device="cuda").manual_seed(M + K)
    A, Bt, B, At = _random(g, M, K), _random(g, N, K), _random(g, K, N), _random(g, K, M)
    d = lambda t: t.double()
    new = lambda *s: torch.full(s, float("nan"), dtype=torch.bfloat16, device="cuda")
    ref = lambda t: t.cpu().numpy()
    # (forward: both operands along the contraction; data gradient: the weight across it; weight gradient: both across it)
    assert_parity(ard.drop_gemm_fwd(A, Bt, out=new(M, N)), ref(d(A) @ d(Bt).t()), "bf16", what="Y")
    assert_parity(ard.drop_gemm_bwd_data(A, B, out=new(M, N)), ref(d(A) @ d(B)), "bf16", what="dX")
    assert_parity(ard.drop_gemm_bwd_weight(At, B, out=new(M, N)), ref(d(At).t() @ d(B)), "bf16", what="dW")


@pytest.mark.parametrize("tile", [32, 64, 128])
@pytest.mark.parametrize("blocks", [3, 8, 13, 18])
def test_tile_pattern_contraction_lengths(tile, blocks):
    """Kept blocks of the contraction that lie dp apart, found one after the other."""
    B, O, I, dp = 2048, 3584, blocks * tile, 2
    g = torch.Generator(device="cuda").manual_seed(tile + blocks)
    X, W, dY = _random(g, B, I), _random(g, O, I), _random(g, B, O)
    pat = ard.Pattern.tile(dp, 2, tile, tile)
    t = torch.arange(O // tile * blocks, device="cuda").reshape(O // tile, blocks)
    mask = ((t + 1 - 2) % dp == 0).double().repeat_interleave(tile, 0).repeat_interleave(tile, 1)
    MW = W.double() * mask
    assert_parity(ard.drop_gemm_fwd(X, W, pat), (X.double() @ MW.t()).cpu().numpy(), "bf16", what="Y")
    assert_parity(ard.drop_gemm_bwd_data(dY, W, pat), (dY.double() @ MW).cpu().numpy(), "bf16", what="dX")
