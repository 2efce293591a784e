"""The iterator that gives the steady loop of the LDS-direct products its places, stepped beside the arithmetic that the bounds proof
walks: plain and block contractions, convolutions and their weight gradients, contractions split anywhere.  Without a GPU."""
import pytest

import dryrun as D


def _compared(lib, rcs, what):
    for rc in rcs:
        assert rc == 0, f"{what}: status {rc}: {lib.ard_last_error().decode()}"
    assert "gemm_direct_kernel" in D.launches(lib)[1], what
    return lib.ard_debug_compared_slabs()


@pytest.mark.parametrize("op", [0, 1, 2])
def test_plain_and_split_contractions(op):
    with D.dry_run() as lib:
        lib.ard_debug_compared_slabs()
        heap = D.FakeHeap()
        for B, I, O in ((2048, 704, 3584), (1024, 2040, 1000), (72, 6144, 64), (64, 72, 6144), (6144, 64, 80), (4096, 200, 200)):
            n = _compared(lib, D.layer_calls(lib, heap, D.BF16, B, I, O, None, None, 0, ops=(op,)), f"{B} {I} {O}")
            steps = -(-(I, O, B)[op] // 64)
            assert n > 0 or steps <= 3, (B, I, O, n)


@pytest.mark.parametrize("tile", [32, 64, 128])
@pytest.mark.parametrize("dp", [1, 2, 3, 5])
def test_kept_blocks_of_the_contraction(tile, dp):
    with D.dry_run() as lib:
        lib.ard_debug_compared_slabs()
        heap = D.FakeHeap()
        for b in {1, dp}:
            for op in (0, 1):
                n = _compared(lib, D.layer_calls(lib, heap, D.BF16, 2048, 32 * tile, 29 * tile, (dp, b), None, 0, tile=(tile, tile), ops=(op,)), f"{tile} {dp} {b}")
                assert n > 0, (tile, dp, b, op)


@pytest.mark.parametrize("k", [1, 3, 5])
@pytest.mark.parametrize("N,Cc,Cout,S,n_keep", [(16, 192, 256, 14, 192), (128, 256, 256, 28, 256), (60, 512, 520, 9, 512), (40, 300, 130, 13, 300)])
def test_taps_and_channel_groups(N, Cc, Cout, S, n_keep, k):
    """Forward, data gradient (steps: every tap of a channel group) and weight gradient (pixels of the grid) of a convolution."""
    with D.dry_run() as lib:
        lib.ard_debug_compared_slabs()
        for mode in (1, 2, 3):
            n = _compared(lib, D.conv_calls(lib, D.FakeHeap(), D.BF16, N, Cc, Cout, S, S, k, 1, k // 2, n_keep, modes=(mode,)), f"{N} {Cc} {k} mode {mode}")
            assert n > 0 or k == 1, (mode, n)
