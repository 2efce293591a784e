"""GPU parity of bf16 tile patterns whose sizes are multiples of nothing (operands copied with padded rows before the
tile-class products): remainders of 1, 4 and 7 on either side, extents below one tile, odd and even row starts of the
outputs, a gradient gated by an activation, beside operands that start at odd addresses and workspaces with room for the
tile lists alone (the general engine takes those)."""
import numpy as np
import pytest
import torch

from oracle import gemm as G
from oracle import patterns as P
from paper_2203_05705_amd import binding as ard
from util import assert_parity, from_vals, stored

pytestmark = pytest.mark.gpu

CASES = [(1, 1, 1, 32, 32, 1, 1), (37, 33, 65, 32, 32, 2, 1), (64, 90, 128, 64, 64, 3, 2), (130, 128, 95, 32, 32, 2, 2), (226, 292, 1269, 32, 32, 2, 1),
         (21, 1423, 384, 64, 64, 1, 1), (1000, 503, 337, 64, 64, 5, 3), (513, 1030, 1001, 32, 64, 8, 8), (96, 2049, 777, 128, 64, 6, 4), (23, 803, 399, 128, 256, 2, 1), (64, 555, 1030, 256, 256, 3, 2)]


def _operands(B, I, O, skew=0):
    rng = np.random.default_rng(B + I + O)
    vals = [stored(rng.standard_normal(s), "bf16") for s in ((B, I), (O, I), (B, O))]
    dev = [from_vals(v, "bf16") for v in vals]
    if skew:
        moved = [torch.empty(t.numel() + skew, dtype=t.dtype, device="cuda") for t in dev]
        dev = [m[skew:].view(t.shape).copy_(t) for m, t in zip(moved, dev)]
    return vals, dev


@pytest.mark.parametrize("B,I,O,x,y,dp,b,how", [c + ("copies",) for c in CASES] + [c + (how,) for c in CASES[1:5] for how in ("no room", "askew")])
def test_ragged_tile_patterns(B, I, O, x, y, dp, b, how):
    print("ragged tiles", B, I, O, x, y, dp, b, how, flush=True)
    (Xv, Wv, dYv), (X, W, dY) = _operands(B, I, O, 1 if how == "askew" else 0)
    MW = P.expand_tile_mask(P.tile_mask(O, I, x, y, dp, b), O, I, x, y).astype(np.float64)
    ones = np.ones(O, np.uint8)
    pat = ard.Pattern.tile(dp, b, x, y)
    lists = ard.gemm_workspace_bytes(ard.F32, B, I, O, pat)
    ws = torch.full((lists if how == "no room" else ard.gemm_workspace_bytes(ard.BF16, B, I, O, pat),), 0xFF, dtype=torch.uint8, device="cuda")
    Y, dX, dW = (torch.full(s, float("nan"), dtype=torch.bfloat16, device="cuda") for s in ((B, O), (B, I), (O, I)))
    ard.drop_gemm_fwd(X, W, pat, alpha=0.5, relu=True, out=Y, ws=ws)
    ard.drop_gemm_bwd_data(dY, W, pat, relu_src=X, out=dX, ws=ws)
    ard.drop_gemm_bwd_weight(dY, X, pat, out=dW, ws=ws)
    assert_parity(Y, np.maximum(G.drop_gemm_fwd(Xv, Wv, MW, ones, 0.5), 0), "bf16", what="Y")
    assert_parity(dX, G.drop_gemm_bwd_data(dYv, Wv, MW, ones) * (Xv > 0), "bf16", what="dX")
    assert_parity(dW, G.drop_gemm_bwd_weight(dYv, Xv, MW, ones), "bf16", zero_mask=(MW == 0), what="dW")


def test_the_static_weight_gradient_takes_what_it_took():
    """A layer whose copies do not fit into the library's own scratch is computed without them."""
    B, I, O = 8191, 2731, 2047
    (Xv, _, dYv), (X, _, dY) = _operands(B, I, O)
    pat = ard.Pattern.tile(8, 1, 64, 64)
    assert ard.gemm_workspace_bytes(ard.BF16, B, I, O, pat) > ard.lib().ard_static_scratch_bytes()
    dW = torch.full((O, I), float("nan"), dtype=torch.bfloat16, device="cuda")
    ard.drop_gemm_bwd_weight_static(dY, X, pat, None, dW)
    ws = torch.empty(ard.gemm_workspace_bytes(ard.BF16, B, I, O, pat), dtype=torch.uint8, device="cuda")
    assert_parity(dW, ard.drop_gemm_bwd_weight(dY, X, pat, ws=ws).float().cpu().numpy().astype(np.float64), "bf16", rounded_ref=True, what="dW")
