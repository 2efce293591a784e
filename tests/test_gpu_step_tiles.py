"""GPU parity of the bf16 products whose tile every case asserts, at every number of contraction steps around the point from which
their loads are spread over the steps: convolutions (steps: filter taps by channel groups) and their weight gradients (pixels of the
grid), tiles of 128 x 128 and 128 x 64, blocks of 32 of a tile pattern.  Reference: the same stored values in 64 bits."""
import pytest
import torch

import dryrun as D
import test_gpu_steps as steps
from paper_2203_05705_amd import binding as ard
from util import assert_parity

pytestmark = pytest.mark.gpu


def _conv_instances(mode, N, C, Cout, S, k):
    with D.dry_run() as lib:
        D.launches(lib)
        assert D.conv_calls(lib, D.FakeHeap(), D.BF16, N, C, Cout, S, S, k, 1, k // 2, C, modes=(mode,)) == [0]
        return D.instances(lib)


def _shifted(A, k):
    """The kept planes as the taps of a k x k filter see them: [taps, N, C, S * S] in 64 bits, one at a time."""
    N, C, S, _ = A.shape
    P = torch.nn.functional.pad(A.double(), (k // 2,) * 4)
    for r in range(k):
        for s in range(k):
            yield r, s, P[:, :, r:r + S, s:s + S].reshape(N, C, S * S).contiguous()


def _layer(N, C, Cout, S, k):
    g = torch.Generator(device="cuda").manual_seed(C + Cout + S)
    new = lambda *s: torch.randn(s, generator=g, device="cuda").to(torch.bfloat16)
    return new(N, C, S, S), new(Cout, C, k, k) * 0.125, new(N, Cout, S, S), torch.arange(C, dtype=torch.int32, device="cuda")


# (two stages of loads in flight: spread from six or seven steps on, three: from eight or nine)
FORWARD = [("128, 448", 128, 128, 28, (5, 6, 7, 8)), ("128, 384", 128, 384, 14, (5, 6, 7, 8)), ("256, 256", 64, 256, 28, (5, 6, 7)),
           ("256, 128", 128, 256, 14, (7, 8, 9, 10)), ("128, 256", 128, 128, 14, (7, 8, 9, 10)), ("64, 64", 33, 100, 14, (6, 7, 8))]


@pytest.mark.parametrize("tile,N,Cout,S,C,k", [(t, N, Co, S, 64 * n, 1) for t, N, Co, S, ns in FORWARD for n in ns]
                         + [(t, N, Co, S, 64 * c, 3) for t, N, Co, S, _ in FORWARD for c in (1, 2)] + [("128, 256", 128, 128, 14, 128, 5)])
def test_convolution(tile, N, Cout, S, C, k):
    assert f"gemm_direct_kernel<{tile}, 1>" in _conv_instances(1, N, C, Cout, S, k)
    A, Wt, _, keep = _layer(N, C, Cout, S, k)
    ref = 0
    for r, s, X in _shifted(A, k):
        ref = ref + torch.matmul(Wt[:, :, r, s].double().contiguous(), X)
    Y = torch.full((N, Cout, S, S), float("nan"), dtype=torch.bfloat16, device="cuda")
    ard.conv_fwd(A, Wt, keep, C, pad=k // 2, out=Y)
    assert_parity(Y, ref.reshape(Y.shape).cpu().numpy(), "bf16", what="Y")


@pytest.mark.parametrize("tile,C,Cout", [("256, 128", 70, 136), ("128, 128", 70, 72)])
@pytest.mark.parametrize("N,S,k", [(1, 7, 3), (2, 13, 3), (9, 14, 3), (33, 14, 1), (57, 9, 5)])
def test_weight_gradient(tile, C, Cout, N, S, k):
    assert f"gemm_direct_kernel<{tile}, 2>" in _conv_instances(3, N, C, Cout, S, k)
    A, _, dY, keep = _layer(N, C, Cout, S, k)
    G = dY.double().reshape(N, Cout, S * S).permute(1, 0, 2).reshape(Cout, N * S * S)
    ref = torch.empty((Cout, C, k, k), dtype=torch.float64, device="cuda")
    for r, s, X in _shifted(A, k):
        ref[:, :, r, s] = G @ X.permute(0, 2, 1).reshape(N * S * S, C)
    dW = torch.full((Cout, C, k, k), float("nan"), dtype=torch.bfloat16, device="cuda")
    ard.conv_bwd_weight(dY, A, keep, C, ksize=(k, k), pad=k // 2, out=dW)
    assert_parity(dW, ref.cpu().numpy(), "bf16", what="dWt")


def _layer_instances(B, I, O, po, pi, op):
    with D.dry_run() as lib:
        D.launches(lib)
        assert D.layer_calls(lib, D.FakeHeap(), D.BF16, B, I, O, po, pi, 0, ops=(op,)) == [0]
        return D.instances(lib)


@pytest.mark.parametrize("n", [2, 3, 4, 5, 6, 7, 8])
@pytest.mark.parametrize("op", [0, 1, 2])
def test_four_wavefront_tiles(op, n):
    """128 x 64: a plain product.  128 x 128: results spread among dropped columns."""
    K = 64 * n + (24 if n % 2 else 0)
    g = torch.Generator(device="cuda").manual_seed(n)
    new = lambda *s: torch.randn(s, generator=g, device="cuda").to(torch.bfloat16)
    for tile, dims, po, pi in (("128, 64", (2048, 2048), None, None), ("128, 128", (2048, 4096), (2, 2), (2, 1))):
        M, N = dims
        # product M x N (of the kept) over K: forward M = B, N = O, K = I; data gradient N = I, K = O; weight gradient M = O, N = I, K = B
        B, I, O = ((M, K, N), (M, N, K), (K, N, M if po is None else 4096))[op]
        fo, fi = po if op != 1 else None, pi if op != 0 else None
        assert any(f"gemm_direct_kernel<{tile}, 0>" == i for i in _layer_instances(B, I, O, fo, fi, op)), _layer_instances(B, I, O, fo, fi, op)
        X, W, dY = new(B, I), new(O, I), new(B, O)
        pat = lambda p: None if p is None else ard.Pattern.row(*p)
        mo, mi = torch.zeros(O, dtype=torch.float64, device="cuda"), torch.zeros(I, dtype=torch.float64, device="cuda")
        mo[slice(None) if fo is None else slice(fo[1] - 1, None, fo[0])] = 1
        mi[slice(None) if fi is None else slice(fi[1] - 1, None, fi[0])] = 1
        nan = lambda *s: torch.full(s, float("nan"), dtype=torch.bfloat16, device="cuda")
        MW = W.double() * mo[:, None] * mi[None, :]
        if op == 0:
            got, ref = ard.drop_gemm_fwd(X, W, pat(fo), pat(fi), out=nan(B, O)), X.double() @ MW.t()
        elif op == 1:
            got, ref = ard.drop_gemm_bwd_data(dY, W, pat(fo), pat(fi), out=nan(B, I)), dY.double() @ MW
        else:
            got, ref = ard.drop_gemm_bwd_weight(dY, X, pat(fo), pat(fi), out=nan(O, I)), (dY.double().t() @ X.double()) * mo[:, None] * mi[None, :]
        assert_parity(got, ref.cpu().numpy(), "bf16", what=f"{tile} op {op}")


@pytest.mark.parametrize("blocks", [26, 29, 30, 31, 32, 46])
def test_blocks_of_32(blocks):
    """Half of the blocks are kept: from seven steps on, two blocks a step and one in the last."""
    steps.test_tile_pattern_contraction_lengths(32, blocks)
