"""GPU parity of the forward pass under the block pattern on tiles of 128 positions that end anywhere in a band (bf16,
stride 1, blocks of whole 64-channel groups), at the sizes where its kernel changes branch: a tile that is not full, tiles over
several images, one output channel and several tiles of 64, one and several groups, a last group that is not full, more
than 64 contraction steps, no kept block at all, planes stored 16, 8, 4 and 2 bytes at a time, paddings that shrink and
grow the image, bands of one position, layers of less than a tile."""
import numpy as np
import pytest
import torch

from dryrun import FakeHeap, dry_run, launches
from oracle import sensitivity as S
from paper_2203_05705_amd import binding as ard
from util import assert_parity, from_vals, stored

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,C,Cout,H,W,k,pad,x,groups,p", [
    (1, 64, 1, 16, 20, 3, 1, 12, 1, 0.5), (7, 64, 16, 7, 7, 3, 1, 12, 1, 0.5), (11, 128, 65, 7, 7, 3, 1, 49, 1, 0.3), (3, 192, 130, 13, 13, 3, 1, 13, 2, 0.4),
    (2, 448, 40, 14, 14, 3, 1, 28, 1, 0.3), (2, 320, 24, 16, 16, 5, 2, 100, 1, 0.3), (3, 100, 72, 12, 12, 3, 1, 17, 1, 0.5), (7, 128, 200, 9, 10, 3, 0, 16, 1, 0.5),
    (3, 64, 33, 8, 12, 3, 2, 20, 1, 0.6), (4, 128, 64, 16, 16, 1, 0, 32, 1, 0.5), (2, 128, 64, 16, 16, 3, 1, 32, 1, 0.0), (2, 128, 64, 16, 16, 3, 1, 32, 1, 1.0),
    (30, 64, 100, 5, 5, 3, 1, 25, 1, 0.4), (1, 64, 1, 3, 3, 3, 1, 1, 1, 0.6), (3, 128, 70, 9, 9, 3, 1, 1, 1, 0.5), (2, 192, 24, 13, 13, 3, 1, 5, 2, 0.4),
    (9, 64, 33, 12, 12, 3, 1, 8, 1, 0.3), (2, 128, 200, 12, 12, 3, 1, 72, 1, 0.4), (3, 100, 140, 12, 13, 3, 1, 78, 1, 0.4), (1, 256, 300, 8, 8, 1, 0, 64, 2, 0.5)])
def test_forward(N, C, Cout, H, W, k, pad, x, groups, p):
    print("blocks forward", N, C, Cout, H, W, k, pad, x, groups, p, flush=True)
    rng = np.random.default_rng(C + H + Cout)
    A, Wt = (stored(rng.standard_normal(s) * 0.5, "bf16") for s in ((N, C, H, W), (Cout, C, k, k)))
    Ad, Wd = from_vals(A, "bf16"), from_vals(Wt, "bf16")
    y = 64 * groups * k * k
    _, RB, CB = ard.sens_regions(A.shape, (k, k), 1, pad, x, y)
    keep = (rng.uniform(size=(N, RB, CB)) < p).astype(np.uint8)
    kd = torch.from_numpy(keep.reshape(-1)).cuda()
    Y = ard.conv_fwd_blocks(Ad, Wd, kd, x, y, 1, pad)
    assert_parity(Y, S.conv_fwd_blocks(A, Wt, keep, x, y, 1, pad), "bf16", None, "Y")
    assert torch.equal(Y, ard.conv_fwd_blocks(Ad, Wd, kd, x, y, 1, pad))


@pytest.mark.parametrize("N,C,Cout,H,W,k,pad,x,cpb,p", [
    (1, 16, 1, 7, 7, 3, 1, 12, 16, 0.5), (3, 64, 24, 13, 13, 3, 1, 52, 64, 0.4), (2, 100, 33, 9, 10, 3, 0, 17, 37, 0.5), (2, 48, 40, 14, 14, 5, 2, 28, 3, 0.3),
    (3, 64, 65, 12, 8, 3, 2, 20, 64, 0.6), (4, 32, 16, 16, 16, 1, 0, 256, 7, 0.5), (2, 128, 64, 16, 16, 3, 1, 32, 64, 0.0), (2, 128, 64, 16, 16, 3, 1, 32, 64, 1.0),
    (2, 40, 16, 10, 10, 3, 1, 30, 2, 0.5), (2, 160, 16, 10, 10, 5, 2, 30, 10, 0.5), (6, 16, 2, 19, 19, 1, 0, 19, 1, 0.5)])
def test_forward_f32(N, C, Cout, H, W, k, pad, x, cpb, p):
    """fp32: one pass per column block, up to 16 of them and the first number beyond, the last with fewer channels, or one over the
    patches of all where blocks are many and small; what no kept block reads does not have to be finite."""
    print("blocks forward f32", N, C, Cout, H, W, k, pad, x, cpb, p, flush=True)
    rng = np.random.default_rng(C + H + Cout)
    A, Wt = (stored(rng.standard_normal(s) * 0.5, "f32") for s in ((N, C, H, W), (Cout, C, k, k)))
    Ad, Wd = from_vals(A, "f32"), from_vals(Wt, "f32")
    y = cpb * k * k
    _, RB, CB = ard.sens_regions(A.shape, (k, k), 1, pad, x, y)
    keep = (rng.uniform(size=(N, RB, CB)) < p).astype(np.uint8)
    keep[0, :, CB - 1] = 0
    Ad[0, (CB - 1) * cpb:] = float("nan")
    Y = ard.conv_fwd_blocks(Ad, Wd, torch.from_numpy(keep.reshape(-1)).cuda(), x, y, 1, pad)
    assert_parity(Y, S.conv_fwd_blocks(A, Wt, keep, x, y, 1, pad), "f32", None, "Y")


@pytest.mark.parametrize("bad", [float("inf"), float("nan")])
@pytest.mark.parametrize("N,C,Cout,H,W,x,groups", [
    (4, 128, 140, 16, 16, 96, 1), (2, 128, 200, 14, 14, 49, 1), (3, 320, 130, 12, 13, 78, 2), (2, 192, 24, 13, 13, 13, 1), (5, 100, 72, 12, 12, 17, 1)])
def test_weights_that_are_not_finite_stay_out_of_dropped_blocks(N, C, Cout, H, W, x, groups, bad):
    """One weight of the second column block that is not finite reaches its output channel where a band keeps that block, and no
    other; a channel all of whose weights are not finite is +0.0 where a band keeps nothing."""
    print("blocks not finite", N, C, Cout, H, W, x, groups, bad, flush=True)
    rng = np.random.default_rng(C + H + Cout)
    A, Wt = (stored(rng.standard_normal(s) * 0.5, "bf16") for s in ((N, C, H, W), (Cout, C, 3, 3)))
    y = 64 * groups * 9
    _, RB, CB = ard.sens_regions(A.shape, (3, 3), 1, 1, x, y)
    keep = (rng.uniform(size=(N, RB, CB)) < 0.5).astype(np.uint8)
    keep[0, 0], keep[N - 1, RB - 1, 1] = 0, 1
    Ad, Wd, kd = from_vals(A, "bf16"), from_vals(Wt, "bf16"), torch.from_numpy(keep.reshape(-1)).cuda()
    clean = ard.conv_fwd_blocks(Ad, Wd, kd, x, y, 1, 1)
    Wd[7, 64 * groups + 5, 1, 1] = bad
    Wd[Cout - 1] = bad
    Y = ard.conv_fwd_blocks(Ad, Wd, kd, x, y, 1, 1).reshape(N, Cout, H * W)
    band = torch.arange(H * W, device="cuda") // x
    kept = torch.from_numpy(keep).cuda().bool()[:, band]   # [N, H * W, CB]
    clean, other = clean.reshape(N, Cout, H * W), torch.ones(Cout, dtype=torch.bool, device="cuda")
    other[[7, Cout - 1]] = False
    assert torch.equal(Y[:, other], clean[:, other])
    assert_parity(Y[:, 7][~kept[:, :, 1]], clean[:, 7][~kept[:, :, 1]].float().cpu().numpy(), "bf16", None, "one weight, dropped", rounded_ref=True)
    assert not torch.isfinite(Y[:, 7][kept[:, :, 1]]).any()
    assert not torch.isfinite(Y[:, Cout - 1][kept.any(-1)]).any()
    assert not Y[:, Cout - 1][~kept.any(-1)].view(torch.int16).any()


def _data_gradient_kernels(N, C, Cout, H, W, k, x, y):
    with dry_run() as lib:
        n, p = lib.ard_conv_workspace_bytes(ard.BF16, N, C, H, W, Cout, k, k, 1, k // 2), FakeHeap()(1 << 20)
        launches(lib)
        assert lib.ard_conv_bwd_blocks(2, ard.BF16, N, C, H, W, Cout, k, k, 1, k // 2, x, y, None, p, p, p, p, p, n, None) == 0
        return launches(lib)[1]


@pytest.mark.parametrize("N,C,Cout,H,W,k,x,groups,p", [
    (4, 64, 48, 16, 36, 7, 144, 1, 0.5), (1, 192, 64, 28, 29, 7, 29, 1, 0.4), (2, 128, 8, 21, 24, 7, 72, 1, 0.5), (9, 512, 40, 31, 27, 3, 81, 2, 0.3),
    (3, 128, 24, 20, 17, 7, 340, 2, 0.5), (2, 192, 24, 20, 21, 7, 147, 1, 0.6), (6, 128, 8, 16, 40, 7, 40, 2, 0.5), (5, 64, 8, 27, 35, 5, 140, 1, 0.5), (2, 128, 100, 29, 39, 7, 273, 1, 0.4),
    (4, 128, 24, 24, 40, 5, 80, 2, 0.0), (4, 128, 24, 24, 40, 5, 80, 2, 1.0)])
def test_data_gradient_over_tiles(N, C, Cout, H, W, k, x, groups, p):
    """Tiles of several bands, one and part of one, one and two groups of 64 channels per block, one and more than 64 steps, planes
    stored 16, 4 and 2 bytes at a time; the weight gradient takes the copy of dY that it leaves."""
    print("blocks data gradient", N, C, Cout, H, W, k, x, groups, p, flush=True)
    rng = np.random.default_rng(C + H + Cout)
    A, Wt, dY = (stored(rng.standard_normal(s) * 0.5, "bf16") for s in ((N, C, H, W), (Cout, C, k, k), (N, Cout, H, W)))
    y = 64 * groups * k * k
    assert "conv_block_data_kernel" in _data_gradient_kernels(N, C, Cout, H, W, k, x, y)
    _, RB, CB = ard.sens_regions(A.shape, (k, k), 1, k // 2, x, y)
    keep = (rng.uniform(size=(N, RB, CB)) < p).astype(np.uint8)
    kd = torch.from_numpy(keep.reshape(-1)).cuda()
    Ad, Wd, dYd = (from_vals(v, "bf16") for v in (A, Wt, dY))
    dA, dW = ard.conv_bwd_blocks(dYd, Ad, Wd, kd, x, y, 1, k // 2)
    # the oracle on the first and the last image
    idx = sorted({0, N - 1})
    rA, _ = S.conv_bwd_blocks(dY[idx], A[idx], Wt, keep[idx], x, y, 1, k // 2)
    assert_parity(dA[idx], rA, "bf16", None, "dA")
    for n in range(0, N, 2):   # (and the weight gradient over all of them, image by image)
        sl = slice(n, min(n + 2, N))
        part = S.conv_bwd_blocks(dY[sl], A[sl], Wt, keep[sl], x, y, 1, k // 2)[1]
        rW = part if n == 0 else rW + part
    assert_parity(dW, rW, "bf16", None, "dWt")
    again, _ = ard.conv_bwd_blocks(dYd, Ad, Wd, kd, x, y, 1, k // 2)
    assert torch.equal(dA, again)


@pytest.mark.parametrize("bad", [float("inf"), float("nan")])
@pytest.mark.parametrize("N,C,Cout,H,W,k,x,groups", [(2, 128, 64, 38, 31, 5, 93, 1), (3, 64, 40, 26, 28, 5, 196, 1), (2, 64, 80, 13, 28, 3, 56, 1)])
def test_data_gradient_with_a_weight_that_is_not_finite(N, C, Cout, H, W, k, x, groups, bad):
    """It reaches the pixels that a kept entry was cut from through its tap, and no other."""
    print("blocks data gradient not finite", N, C, Cout, H, W, k, x, groups, bad, flush=True)
    rng = np.random.default_rng(C + H + Cout)
    Wt, dY = (stored(rng.standard_normal(s) * 0.5, "bf16") for s in ((Cout, C, k, k), (N, Cout, H, W)))
    y = 64 * groups * k * k
    kernels = _data_gradient_kernels(N, C, Cout, H, W, k, x, y)
    assert ("conv_block_data_kernel" if k > 3 else "conv_scatter_data_kernel") in kernels, kernels
    _, RB, CB = ard.sens_regions((N, C, H, W), (k, k), 1, k // 2, x, y)
    keep = (rng.uniform(size=(N, RB, CB)) < 0.5).astype(np.uint8)
    keep[0, 0], keep[N - 1, 0] = 0, 1
    Wd, dYd, kd = from_vals(Wt, "bf16"), from_vals(dY, "bf16"), torch.from_numpy(keep.reshape(-1)).cuda()
    Ad = torch.zeros((N, C, H, W), dtype=torch.bfloat16, device="cuda")
    clean, _ = ard.conv_bwd_blocks(dYd, Ad, Wd, kd, x, y, 1, k // 2)
    c, r, s = C - 3, 0, k - 1
    Wd[5, c, r, s] = bad
    dA, _ = ard.conv_bwd_blocks(dYd, Ad, Wd, kd, x, y, 1, k // 2)
    kept = keep[:, np.arange(H * W) // x, c // (64 * groups)].reshape(N, H, W).astype(bool)
    hit = np.zeros((N, H, W), dtype=bool)   # pixel (h, w) is entry (r, s) of the patch of (h + k // 2 - r, w + k // 2 - s)
    for h in range(H):
        for w in range(W):
            oh, ow = h + k // 2 - r, w + k // 2 - s
            if 0 <= oh < H and 0 <= ow < W:
                hit[:, h, w] = kept[:, oh, ow]
    hit = torch.from_numpy(hit).cuda()
    others = [i for i in range(C) if i != c]
    assert torch.equal(dA[:, others], clean[:, others])
    assert not torch.isfinite(dA[:, c][hit]).any()
    assert_parity(dA[:, c][~hit], clean[:, c][~hit].float().cpu().numpy(), "bf16", None, "pixels it does not reach", rounded_ref=True)
