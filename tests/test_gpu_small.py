"""GPU parity of the small bf16 products in the caller's own layout: sizes around the 32 x 32 tiles, the slices of 32 and the
wavefronts' shares of the contraction, every step the wide loads know and one they do not, odd row starts, operands at odd and at
2-byte aligned addresses, values that are not finite next to the clamped rows and the clamped end of the contraction."""
import numpy as np
import pytest
import torch

from dryrun import FakeHeap, dry_run, launches, layer_calls
from oracle import gemm as G
from oracle import patterns as P
from paper_2203_05705_amd import binding as ard
from util import assert_parity, from_vals, stored

SIZES = [(1, 1, 1), (31, 33, 65), (32, 64, 96), (33, 66, 131), (64, 255, 100), (17, 379, 317), (130, 77, 290), (257, 130, 67)]
STEPS = [(1, 1), (2, 1), (1, 2), (3, 3), (4, 2), (2, 4), (5, 3), (8, 8), (9, 5)]


def _layer(B, I, O, skew=0):
    rng = np.random.default_rng(7 * B + 3 * I + O)
    vals = [stored(rng.standard_normal(s), "bf16") for s in ((B, I), (O, I), (B, O))]
    dev = [from_vals(v, "bf16") for v in vals]
    if skew:
        moved = [torch.empty(t.numel() + skew, dtype=t.dtype, device="cuda") for t in dev]
        dev = [m[skew:].view(t.shape).copy_(t) for m, t in zip(moved, dev)]
    return vals, dev


def _guarded(shape, skew):
    """NaN-filled output inside a buffer of sevens, `skew` elements from an aligned address."""
    n = int(np.prod(shape))
    buf = torch.full((64 + n + 64,), 7.0, dtype=torch.bfloat16, device="cuda")
    out = buf[64 + skew:64 + skew + n]
    out.fill_(float("nan"))
    return buf, out.view(shape), (64 + skew, n)


def _intact(buf, at, n):
    return bool((buf[:at] == 7).all()) and bool((buf[at + n:] == 7).all())


@pytest.mark.gpu
@pytest.mark.parametrize("skew", [0, 1, 2])
@pytest.mark.parametrize("dp,dp_in", STEPS)
@pytest.mark.parametrize("B,I,O", SIZES)
def test_small_layers(B, I, O, dp, dp_in, skew):
    print("small layer", B, I, O, dp, dp_in, skew, flush=True)
    dp, dp_in = min(dp, O), min(dp_in, I)
    (Xv, Wv, dYv), (X, W, dY) = _layer(B, I, O, skew)
    for b, b_in in {(1, 1), (dp, dp_in)}:
        mo, mi = P.row_mask(O, dp, b), P.row_mask(I, dp_in, b_in)
        MW = G.weight_mask_rows(mo, mi)
        po, pi = ard.Pattern.row(dp, b), ard.Pattern.row(dp_in, b_in) if dp_in > 1 else None
        (by, Y, ay), (bx, dX, ax), (bw, dW, aw) = (_guarded(s, skew) for s in ((B, O), (B, I), (O, I)))
        ard.drop_gemm_fwd(X, W, po, pi, alpha=0.5, relu=True, out=Y)
        ard.drop_gemm_bwd_data(dY, W, po, pi, relu_src=X, out=dX)
        ard.drop_gemm_bwd_weight(dY, X, po, pi, out=dW)
        assert _intact(by, *ay) and _intact(bx, *ax) and _intact(bw, *aw)
        assert_parity(Y, np.maximum(G.drop_gemm_fwd(Xv, Wv, MW, mo, 0.5), 0), "bf16", (mo == 0)[None, :], "Y")
        assert_parity(dX, G.drop_gemm_bwd_data(dYv, Wv, MW, mo) * (Xv > 0), "bf16", (mi == 0)[None, :], "dX")
        assert_parity(dW, G.drop_gemm_bwd_weight(dYv, Xv, MW, mo), "bf16", MW == 0, "dW")


@pytest.mark.gpu
@pytest.mark.parametrize("bad", [float("inf"), float("nan")])
def test_dropped_and_last_elements_that_are_not_finite(bad):
    """What is dropped reaches no kept result, and the last row reaches its own results only."""
    B, I, O, dp, dp_in = 33, 131, 70, 3, 2
    (Xv, Wv, dYv), (X, W, dY) = _layer(B, I, O)
    po, pi = ard.Pattern.row(dp, 2), ard.Pattern.row(dp_in, 1)
    mo, mi = P.row_mask(O, dp, 2), P.row_mask(I, dp_in, 1)
    MW = G.weight_mask_rows(mo, mi)
    X[:, torch.from_numpy(mi == 0).cuda()] = bad
    dY[:, torch.from_numpy(mo == 0).cuda()] = bad
    W[torch.from_numpy(MW == 0).cuda()] = bad
    X[B - 1, I - 1], dY[B - 1, 1] = bad, bad
    Y = ard.drop_gemm_fwd(X, W, po, pi)
    dX = ard.drop_gemm_bwd_data(dY, W, po, pi)
    assert_parity(Y[:B - 1], G.drop_gemm_fwd(Xv, Wv, MW, mo)[:B - 1], "bf16", (mo == 0)[None, :], "Y")
    assert_parity(dX[:B - 1], G.drop_gemm_bwd_data(dYv, Wv, MW, mo)[:B - 1], "bf16", (mi == 0)[None, :], "dX")
    assert not torch.isfinite(Y[B - 1, torch.from_numpy(mo == 1).cuda()]).any()
    assert not torch.isfinite(dX[B - 1, torch.from_numpy(mi == 1).cuda()]).any()
    assert bool((dX[:, torch.from_numpy(mi == 0).cuda()] == 0).all())


def test_small_layers_take_one_launch_a_product():
    with dry_run() as lib:
        for B, I, O, po, pi in ((64, 100, 130, (2, 1), (3, 2)), (33, 1024, 513, (8, 8), (2, 1))):
            launches(lib)
            assert layer_calls(lib, FakeHeap(), ard.BF16, B, I, O, po, pi, 0) == [0, 0, 0]
            n, names = launches(lib)
            assert names[-3:] == ["gemm_small_kernel"] * 3, names
        # without the room that a call with an input pattern asks for it is refused as ever
        assert layer_calls(lib, FakeHeap(), ard.BF16, 64, 100, 130, (2, 1), (3, 2), 0, ws_bytes=16, ops=(0,)) != [0]


@pytest.mark.gpu
@pytest.mark.parametrize("grouped", [False, True])
@pytest.mark.parametrize("dp,dp_in", [(1, 1), (1, 3), (2, 2), (3, 1), (5, 4), (8, 6)])
@pytest.mark.parametrize("B,I,O", [(1, 9, 17), (33, 131, 70), (64, 333, 113), (150, 1030, 40)])
def test_compact_activations(B, I, O, dp, dp_in, grouped):
    """Compact activations beside a weight in its own layout, or a compact one: alone and as one grid."""
    print("small compact", B, I, O, dp, dp_in, grouped, flush=True)
    (Xv, Wv, dYv), (X, W, dY) = _layer(B, I, O)
    b, b_in = dp, (dp_in + 1) // 2
    mo, mi = P.row_mask(O, dp, b), P.row_mask(I, dp_in, b_in)
    MW = G.weight_mask_rows(mo, mi)
    ko, ki = np.flatnonzero(mo), np.flatnonzero(mi)
    po, pi = (ard.Pattern.row(dp, b) if dp > 1 else None), (ard.Pattern.row(dp_in, b_in) if dp_in > 1 else None)
    Xc, dYc = ard.pad_compact(X[:, ki].contiguous()), ard.pad_compact(dY[:, ko].contiguous())
    Wc = ard.compact_weight(W, po, pi)
    ws = [torch.full((ard.gemm_workspace_bytes(ard.BF16, B, I, O, po, pi),), 0xFF, dtype=torch.uint8, device="cuda") for _ in range(4)]
    both = ard.IN_COMPACT | ard.OUT_COMPACT
    (bw, dW, aw) = _guarded((O, I), 0)

    def calls():
        return (ard.drop_gemm_fwd(Xc, W, po, pi, relu=True, flags=both, I=I, O=O, ws=ws[0]),
                ard.drop_gemm_bwd_data(dYc, W, po, pi, relu_src=Xc, flags=both, I=I, O=O, ws=ws[1]),
                ard.drop_gemm_fwd(Xc, Wc, po, pi, flags=ard.IN_COMPACT | ard.W_COMPACT, I=I, O=O, ws=ws[2]),
                ard.drop_gemm_bwd_weight(dYc, Xc, po, pi, flags=both, I=I, O=O, out=dW, ws=ws[3]))
    if grouped:
        with ard.batch():
            Yc, dXc, Y, _ = calls()
    else:
        Yc, dXc, Y, _ = calls()
    assert _intact(bw, *aw)
    assert_parity(dW, G.drop_gemm_bwd_weight(dYv, Xv, MW, mo), "bf16", MW == 0, "dW")
    Yr, dXr = G.drop_gemm_fwd(Xv, Wv, MW, mo), G.drop_gemm_bwd_data(dYv, Wv, MW, mo)
    assert_parity(Yc[:, :len(ko)].contiguous(), np.maximum(Yr, 0)[:, ko], "bf16", None, "Y compact")
    assert_parity(dXc[:, :len(ki)].contiguous(), (dXr * (Xv > 0))[:, ki], "bf16", None, "dX compact")
    assert_parity(Y, Yr, "bf16", (mo == 0)[None, :], "Y")
    assert not Yc[:, len(ko):].any() and not dXc[:, len(ki):].any()


@pytest.mark.gpu
@pytest.mark.parametrize("dp,dp_in", [(1, 1), (1, 2), (1, 3), (1, 4), (3, 1), (1, 6)])
def test_grouped_results_are_those_of_the_calls_alone(dp, dp_in):
    """Four wavefronts with two sums each (grouped) and eight with one (alone; four, where there are more than 256 tiles and at
    most four slices): contractions that end in each of the eight sums, with whole slices of 32 and with a part of one."""
    for B, k, N in [(40, 32 * s + t, 70) for s in (1, 2, 3, 5, 7, 8, 9, 12, 16, 17, 21, 31) for t in (0, 9)] + [(600, 100, 520), (520, 128, 600)]:
        print("small grouped", B, k, N, dp, dp_in, flush=True)
        I, O = k * dp_in, N * dp   # (k kept inputs in the forward pass, N kept outputs)
        _, (X, W, dY) = _layer(B, I, O)
        po, pi = (ard.Pattern.row(dp, dp) if dp > 1 else None), (ard.Pattern.row(dp_in, 1) if dp_in > 1 else None)
        with dry_run() as lib:
            launches(lib)
            layer_calls(lib, FakeHeap(), ard.BF16, B, I, O, (dp, dp) if dp > 1 else None, (dp_in, 1) if dp_in > 1 else None, ard.IN_COMPACT | ard.OUT_COMPACT)
            assert launches(lib)[1].count("gemm_small_kernel") >= (3 if dp_in > 1 and k <= 544 else 0)
        kept = lambda M, d, b: ard.pad_compact(M[:, b - 1::d].contiguous())
        Xc, dYc = kept(X, dp_in, 1), kept(dY, dp, dp)
        Wc = ard.compact_weight(W, po, pi)
        ws = [torch.full((ard.gemm_workspace_bytes(ard.BF16, B, I, O, po, pi),), 0xFF, dtype=torch.uint8, device="cuda") for _ in range(4)]
        both = ard.IN_COMPACT | ard.OUT_COMPACT
        dW = [torch.full((O, I), float("nan"), dtype=torch.bfloat16, device="cuda") for _ in range(2)]

        def calls(i):
            return (ard.drop_gemm_fwd(Xc, W, po, pi, relu=True, flags=both, I=I, O=O, ws=ws[0]),
                    ard.drop_gemm_bwd_data(dYc, W, po, pi, relu_src=Xc, flags=both, I=I, O=O, ws=ws[1]),
                    ard.drop_gemm_fwd(Xc, Wc, po, pi, flags=ard.IN_COMPACT | ard.W_COMPACT, I=I, O=O, ws=ws[2]),
                    ard.drop_gemm_bwd_weight(dYc, Xc, po, pi, flags=both, I=I, O=O, out=dW[i], ws=ws[3]))
        alone = calls(0)
        with ard.batch():
            grouped = calls(1)
        for name, a, g in zip(("Y compact", "dX compact", "Y", "dW"), alone, grouped):
            assert torch.equal(a, g), (name, B, I, O)


FAR = [(8, 1192, 1544, 48, 64), (33, 776, 1030, 64, 3), (40, 2304, 96, 1, 24), (17, 130, 3001, 32, 2), (600, 640, 1280, 16, 16)]


@pytest.mark.gpu
@pytest.mark.parametrize("B,I,O,dp,dp_in", FAR)
def test_neurons_far_apart(B, I, O, dp, dp_in):
    """Steps of up to 64, on either side of the line behind which copies and a finishing pass are faster."""
    print("small far apart", B, I, O, dp, dp_in, flush=True)
    (Xv, Wv, dYv), (X, W, dY) = _layer(B, I, O)
    for b, b_in in ((1, 1), (dp, dp_in)):
        mo, mi = P.row_mask(O, dp, b), P.row_mask(I, dp_in, b_in)
        MW = G.weight_mask_rows(mo, mi)
        po, pi = (ard.Pattern.row(dp, b) if dp > 1 else None), (ard.Pattern.row(dp_in, b_in) if dp_in > 1 else None)
        assert_parity(ard.drop_gemm_fwd(X, W, po, pi), G.drop_gemm_fwd(Xv, Wv, MW, mo), "bf16", (mo == 0)[None, :], "Y")
        assert_parity(ard.drop_gemm_bwd_data(dY, W, po, pi), G.drop_gemm_bwd_data(dYv, Wv, MW, mo), "bf16", (mi == 0)[None, :], "dX")
        assert_parity(ard.drop_gemm_bwd_weight(dY, X, po, pi), G.drop_gemm_bwd_weight(dYv, Xv, MW, mo), "bf16", MW == 0, "dW")


def test_which_products_of_neurons_far_apart_are_one_launch():
    with dry_run() as lib:
        got = []
        for B, I, O, dp, dp_in in FAR:
            for op in range(3):
                launches(lib)
                assert layer_calls(lib, FakeHeap(), ard.BF16, B, I, O, (dp, dp) if dp > 1 else None, (dp_in, 1) if dp_in > 1 else None, 0, ops=(op,)) == [0]
                got.append(launches(lib)[1] == ["gemm_small_kernel"])
        assert got == [True, True, False, True, True, False, True, True, True, True, True, False, True, True, False], got
