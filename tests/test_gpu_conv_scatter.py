"""GPU parity of the data gradient that runs over the kept positions of dY (bf16, filters that keep the image's size), at
the sizes where its kernel changes branch: several images, one image and a band of rows per workgroup; no kept position, one,
a tile of 16, 64 per wavefront, more than one round of 256; passes of 64 to 256 channels, one and several; channels that
are and are not whole groups of 16; planes stored 16, 8, 4 and 2 bytes at a time."""
import numpy as np
import pytest
import torch

from dryrun import FakeHeap, dry_run, launches
from oracle import sensitivity as S
from paper_2203_05705_amd import binding as ard
from util import assert_parity, from_vals, stored

pytestmark = pytest.mark.gpu


def _layer(N, C, Cout, H, W, k, seed):
    rng = np.random.default_rng(seed)
    vals = [stored(rng.standard_normal(s) * 0.5, "bf16") for s in ((N, C, H, W), (Cout, C, k, k), (N, Cout, H, W))]
    return rng, vals, [from_vals(v, "bf16") for v in vals]


@pytest.mark.parametrize("N,C,Cout,H,W,k,p", [
    (1, 1, 65, 1, 1, 1, 1.0), (3, 16, 72, 7, 7, 3, 0.0), (2, 17, 72, 7, 7, 3, 0.02), (70, 200, 66, 7, 7, 3, 0.3), (2, 20, 64, 7, 7, 3, 0.3), (70, 130, 72, 5, 9, 3, 1.0),
    (9, 48, 130, 14, 14, 5, 0.5), (2, 40, 256, 28, 28, 3, 0.3), (64, 256, 200, 28, 28, 3, 1.0), (3, 20, 320, 13, 13, 3, 0.6), (2, 33, 600, 19, 11, 3, 0.7),
    (5, 64, 40, 56, 56, 3, 0.3), (2, 500, 16, 32, 32, 3, 0.8), (2, 24, 64, 12, 100, 3, 0.4), (4, 32, 24, 30, 30, 1, 0.5), (1, 16, 72, 4, 500, 3, 0.5), (1, 16, 72, 4, 900, 3, 0.5),
    (1, 600, 24, 17, 16, 7, 0.5)])
def test_row_pattern(N, C, Cout, H, W, k, p):
    print("rows", N, C, Cout, H, W, k, p, flush=True)
    rng, (A, Wt, dY), (Ad, Wd, dYd) = _layer(N, C, Cout, H, W, k, C + H)
    mask = (rng.uniform(size=(N, H * W)) < p).astype(np.uint8)
    pat = dict(mask=torch.from_numpy(mask.reshape(-1)).cuda())
    dA, _ = ard.conv_bwd_rows(dYd, Ad, Wd, pat, 1, k // 2)
    again, _ = ard.conv_bwd_rows(dYd, Ad, Wd, pat, 1, k // 2)
    # the oracle on the first, a middle and the last image
    idx = sorted({0, N // 2, N - 1})
    ref, _ = S.conv_bwd_rows(dY[idx], A[idx], Wt, mask[idx], 1, k // 2)
    assert_parity(dA[idx], ref, "bf16", None, "dA")
    assert torch.equal(dA, again), "two calls differ"


@pytest.mark.parametrize("N,C,Cout,H,W,k,x,group", [
    (2, 64, 16, 13, 13, 3, 5, 16), (3, 96, 130, 16, 16, 3, 100, 32), (2, 80, 24, 28, 28, 3, 56, 48), (40, 48, 256, 7, 7, 3, 49, 16), (2, 130, 40, 20, 12, 5, 7, 64), (2, 64, 8, 39, 40, 5, 100, 64)])
def test_block_pattern(N, C, Cout, H, W, k, x, group):
    """Column blocks of 16 and more channels, the last one smaller; bands that end anywhere in a row.  (The last layer's one column
    block takes a pass over all positions of a masked copy, which the weight gradient shares.)"""
    print("blocks", N, C, Cout, H, W, k, x, group, flush=True)
    rng, (A, Wt, dY), (Ad, Wd, dYd) = _layer(N, C, Cout, H, W, k, C + x)
    y = group * k * k
    _, RB, CB = ard.sens_regions(A.shape, (k, k), 1, k // 2, x, y)
    keep = (rng.uniform(size=(N, RB, CB)) < 0.4).astype(np.uint8)
    dA, dW = ard.conv_bwd_blocks(dYd, Ad, Wd, torch.from_numpy(keep.reshape(-1)).cuda(), x, y, 1, k // 2)
    rA, rW = S.conv_bwd_blocks(dY, A, Wt, keep, x, y, 1, k // 2)
    assert_parity(dA, rA, "bf16", None, "dA")
    assert_parity(dW, rW, "bf16", None, "dWt")


def test_an_infinity_stays_where_it_belongs():
    """An infinity in a dropped position of dY reaches nothing, one in a kept position the 3 x 3 window around it."""
    N, C, Cout, H = 2, 32, 40, 9
    rng, (A, Wt, dY), (Ad, Wd, dYd) = _layer(N, C, Cout, H, H, 3, 5)
    mask = (rng.uniform(size=(N, H, H)) < 0.5).astype(np.uint8)
    mask[0, 4, 4], mask[1, 2, 2] = 1, 0
    dYd[0, 7, 4, 4] = float("inf")
    dYd[1, 3, 2, 2] = float("inf")
    dA, _ = ard.conv_bwd_rows(dYd, Ad, Wd, dict(mask=torch.from_numpy(mask.reshape(-1)).cuda()), 1, 1)
    bad = ~torch.isfinite(dA.float())
    assert bad[0, :, 3:6, 3:6].all()
    bad[0, :, 3:6, 3:6] = False
    assert not bad.any()


@pytest.mark.parametrize("N,C,Cout,S_,share", [(16, 448, 127, 16, 0.3), (16, 448, 127, 16, 1.0), (40, 256, 200, 28, 0.3), (40, 256, 200, 28, 1.0)])
def test_the_number_of_kept_rows_only_chooses(N, C, Cout, S_, share):
    """The gradient of FWD_ROWS with its number of kept rows, without it and with a number that cannot be: the same sums."""
    print("rows hint", N, C, Cout, S_, share, flush=True)
    rng, (_, Wt, dY), (_, Wd, dYd) = _layer(N, C, Cout, S_, S_, 3, C)
    mask = (rng.uniform(size=(N, S_ * S_)) < share).astype(np.uint8)
    md = torch.from_numpy(mask.reshape(-1)).cuda()
    used = []
    for n_keep in (int(mask.sum()), 0, -5, N * S_ * S_ + 1):
        with dry_run() as lib:
            n, p = lib.ard_conv_workspace_bytes(ard.BF16, N, C, S_, S_, Cout, 3, 3, 1, 1), FakeHeap()(1 << 20)
            launches(lib)
            assert lib.ard_fmap_drop_conv(5, ard.BF16, N, C, S_, S_, Cout, 3, 3, 1, 1, 0.0, n_keep, None, p, p, p, p, None, None, None, p, n, None) == 0
            used.append("conv_scatter_data_kernel" in launches(lib)[1])
        dA = torch.full((N, C, S_, S_), float("nan"), dtype=torch.bfloat16, device="cuda")
        ard.fmap_drop_conv(5, (N, C, S_, S_), ard.BF16, Cout, (3, 3), 1, 1, n_keep=n_keep, Wt=Wd, dY=dYd, out=dA, mask=md)
        idx = [0, N - 1]
        ref, _ = S.conv_bwd_rows(dY[idx], np.zeros((2, C, S_, S_)), Wt, mask[idx], 1, 1)
        assert_parity(dA[idx], ref, "bf16", None, "dA")
    assert used[1] == used[2] == used[3] and used[0] == (share < 0.5)
