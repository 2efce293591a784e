"""Host-side bounds proof of the LDS-direct loaders, without a GPU.

In dry-run mode every entry point runs its dispatch and, for each launch that fetches operands with
unchecked per-lane addresses, walks every workgroup, wavefront, lane and contraction step with the
kernel's own address arithmetic and checks the bytes touched against the operand's extent.  These
tests push the benchmark configurations and the seeded random generators of the GPU tests through it."""
import numpy as np
import pytest

import dryrun as D
from paper_2203_05705_amd import binding as ard

IN, OUT, WC, DW = ard.IN_COMPACT, ard.OUT_COMPACT, ard.W_COMPACT, ard.DW_COMPACT


def _ok(lib, rcs, what):
    for rc in rcs:
        assert rc == 0, f"{what}: status {rc}: {lib.ard_last_error().decode()}"


def test_dry_run_launches_nothing_and_reports_kernels():
    with D.dry_run() as lib:
        heap = D.FakeHeap()
        _ok(lib, D.layer_calls(lib, heap, D.BF16, 1024, 2048, 2048, (2, 1), (2, 2), IN | OUT), "layer")
        n, names = D.launches(lib)
        assert n >= 3 and "gemm_direct_kernel" in names
        n_proofs, six = D.last_bounds(lib)
        assert n_proofs >= 3
        a_lo, a_hi, a_bytes, b_lo, b_hi, b_bytes = six
        assert 0 <= a_lo < a_hi <= a_bytes and 0 <= b_lo < b_hi <= b_bytes


def test_config2_all_pattern_pairs():
    """MLP 784-2048-2048-10 at batch 1024: the nine calls of an iteration for all 64 (dp1, dp2)."""
    with D.dry_run() as lib:
        heap = D.FakeHeap()
        proofs = 0
        for dp1 in range(1, 9):
            for dp2 in range(1, 9):
                p1, p2 = (dp1, 1 + (dp1 * 3 + dp2) % dp1), (dp2, 1 + (dp1 + dp2 * 5) % dp2)
                w = f"pair {p1} {p2}"
                _ok(lib, D.layer_calls(lib, heap, D.BF16, 1024, 784, 2048, p1, None, OUT, ops=(0, 2)), w + " L1")
                _ok(lib, D.layer_calls(lib, heap, D.BF16, 1024, 2048, 2048, p2, p1, IN | OUT), w + " L2")
                _ok(lib, D.layer_calls(lib, heap, D.BF16, 1024, 2048, 2048, p2, p1, IN | OUT | WC, ops=(0, 1)), w + " L2c")
                _ok(lib, D.layer_calls(lib, heap, D.BF16, 1024, 2048, 10, None, p2, IN | OUT), w + " L3")
                proofs += D.last_bounds(lib)[0]
        assert proofs >= 64 * 5


@pytest.mark.parametrize("dp", range(1, 9))
def test_config3_tile_patterns(dp):
    with D.dry_run() as lib:
        heap = D.FakeHeap()
        for b in range(1, dp + 1):
            _ok(lib, D.layer_calls(lib, heap, D.BF16, 4096, 4096, 4096, (dp, b), None, 0, tile=(64, 64)), f"dp={dp} b={b}")
        assert D.last_bounds(lib)[0] >= 1


def test_random_layers_and_tile_patterns():
    from test_gpu_random_shapes import draw_case, draw_tile_case
    with D.dry_run() as lib:
        heap = D.FakeHeap()
        for seed in range(40):
            rng = np.random.default_rng(1000 + seed)
            for _ in range(5):
                B, I, O, po, pi = draw_case(rng)
                for flags in (0, IN | OUT, IN | OUT | WC, IN, OUT, IN | OUT | DW):
                    _ok(lib, D.layer_calls(lib, heap, D.BF16, B, I, O, po, pi, flags), f"layer {B} {I} {O} {po} {pi} {flags}")
        for seed in range(60):
            B, I, O, x, y, dp, b = draw_tile_case(np.random.default_rng(2000 + seed))
            _ok(lib, D.layer_calls(lib, heap, D.BF16, B, I, O, (dp, b), None, 0, tile=(x, y)), f"tile {B} {I} {O} {x}x{y} {dp},{b}")
        assert D.last_bounds(lib)[0] > 100


def test_ragged_tile_patterns():
    """Copies with padded rows: every remainder of either side modulo 8, extents below, at and beyond whole tiles."""
    with D.dry_run() as lib:
        heap = D.FakeHeap()
        for i in range(48):
            I, O = 61 + i % 8 + 96 * (i % 5), 57 + i // 3 % 8 + 64 * (i % 7)
            x, y = ((32, 32), (64, 64), (32, 64), (128, 64))[i % 4]
            dp = 1 + i % min(8, -(-O // x) * -(-I // y))
            _ok(lib, D.layer_calls(lib, heap, D.BF16, 1 + 37 * (i % 11), I, O, (dp, 1 + i % dp), None, 0, tile=(x, y)), f"ragged {I} {O} {x}x{y} {dp}")
            _, names = D.launches(lib)
            assert "gemm_direct_kernel" in names and "gemm_kernel" not in names, names
        assert D.last_bounds(lib)[0] > 48


def test_ragged_tile_weight_gradients_of_few_rows_in_few_large_tiles():
    """Rows that start at odd elements, tiles of 256 columns: up to 63 rows and 32 tiles on the general engine."""
    with D.dry_run() as lib:
        heap = D.FakeHeap()
        for (B, I, O, x, dp), general in (((23, 803, 399, 128, 2), True), ((64, 803, 399, 128, 2), False), ((23, 804, 399, 128, 2), False), ((23, 8003, 3999, 256, 2), False)):
            D.launches(lib)
            _ok(lib, D.layer_calls(lib, heap, D.BF16, B, I, O, (dp, 1), None, 0, tile=(x, 256), ops=(2,)), f"ragged {B} {I} {O}")
            assert ("gemm_kernel" in D.launches(lib)[1]) == general, (B, I, O)


def test_the_shape_that_faulted_once():
    """W 2480 x 2760 with 256-row tiles: the last tile row holds 176 rows (block axes are clamped)."""
    with D.dry_run() as lib:
        heap = D.FakeHeap()
        _ok(lib, D.layer_calls(lib, heap, D.BF16, 1965, 2760, 2480, (7, 1), None, 0, tile=(256, 64)), "256x64")
        _ok(lib, D.layer_calls(lib, heap, D.BF16, 968, 1864, 3144, (3, 3), None, 0, tile=(256, 128)), "256x128")


def test_lstm_and_conv_shapes():
    with D.dry_run() as lib:
        heap = D.FakeHeap()
        for T, B, I, H, dp, b in [(64, 128, 1024, 1024, 2, 2), (64, 128, 1024, 1024, 1, 1), (64, 128, 1024, 1024, 3, 1),
                                  (5, 6, 24, 32, 2, 1), (4, 3, 10, 37, 3, 3), (3, 70, 40, 64, 1, 1), (6, 33, 72, 136, 4, 2),
                                  (3, 64, 128, 200, 3, 1), (35, 20, 1500, 1500, 2, 1)]:
            _ok(lib, D.lstm_calls(lib, heap, D.BF16, T, B, I, H, (dp, b)), f"lstm {T} {B} {I} {H} {dp}")
        n_lstm = D.last_bounds(lib)[0]
        for N, Cc, Cout, H, W, k, pad, nk in [(128, 256, 256, 28, 28, 3, 1, 128), (128, 256, 256, 28, 28, 3, 1, 256),
                                              (2, 8, 16, 7, 7, 3, 1, 4), (3, 12, 20, 9, 6, 3, 1, 8), (2, 16, 8, 8, 8, 1, 0, 12),
                                              (2, 6, 10, 11, 10, 5, 2, 3), (5, 24, 130, 10, 12, 3, 1, 6), (7, 70, 300, 13, 17, 3, 1, 65),
                                              (3, 16, 24, 12, 12, 3, 0, 8), (2, 8, 8, 9, 7, 5, 1, 8),
                                              # few output positions: small tiles for many output channels
                                              (128, 512, 512, 7, 7, 3, 1, 256), (128, 512, 512, 14, 14, 3, 1, 256),
                                              (4, 64, 300, 7, 7, 3, 1, 64), (64, 128, 128, 56, 56, 3, 1, 64)]:
            modes = (1, 2, 3, 0x101, 0x202, 0x103) + ((0x303,) if k - 1 == 2 * pad else ())   # with and without shared grids
            _ok(lib, D.conv_calls(lib, heap, D.BF16, N, Cc, Cout, H, W, k, 1, pad, nk, modes=modes), f"conv {N} {Cc} {Cout} {H}x{W} k{k} keep {nk}")
        assert n_lstm >= 10 and D.last_bounds(lib)[0] >= 10 * 3
        # forward over a list of kept output positions (row-based sensitivity-aware pattern): the list lives in
        # device memory, the proof takes its two extreme readings
        for N, Cc, Cout, H, W, k, pad, rows_kept in [(128, 256, 256, 28, 28, 3, 1, 50000), (2, 8, 16, 7, 7, 3, 1, 40),
                                                       (5, 24, 130, 10, 12, 3, 1, 1), (3, 12, 20, 9, 6, 3, 1, 162)]:
            _ok(lib, D.conv_calls(lib, heap, D.BF16, N, Cc, Cout, H, W, k, 1, pad, rows_kept, modes=(4,)), f"rows {N} {Cc} {H}x{W}")
        assert D.last_bounds(lib)[0] == 4


def test_block_pattern_dispatch_and_bounds():
    """Forward pass under the block pattern: blocks of whole 64-channel groups over all taps with bands of at
    least half a tile, from 256 tiles on, go to the LDS-direct kernel (tile plan in the copy's launch, per-tile block lists,
    proof over the whole contraction), those of fewer tiles or shorter bands to the kernel whose tiles end anywhere in a
    band; any other block shape goes to the general engine."""
    PLAN, ANYWHERE, GENERAL = "gemm_direct_kernel", "conv_block_fwd_kernel", "conv_gemm_kernel"
    with D.dry_run() as lib:
        heap = D.FakeHeap()
        for (N, Cc, Cout, H, W, k, pad, x, y), engine in [((128, 256, 256, 28, 28, 3, 1, 112, 576), PLAN),
                                                           ((128, 256, 256, 28, 28, 3, 1, 196, 1152), PLAN),
                                                           ((128, 128, 200, 12, 12, 3, 1, 72, 576), PLAN),
                                                           ((128, 100, 140, 12, 13, 3, 1, 78, 576), PLAN),
                                                           ((256, 100, 100, 12, 13, 3, 1, 156, 576), PLAN),
                                                           ((256, 192, 130, 9, 16, 3, 1, 144, 0), PLAN),
                                                           ((2, 128, 200, 12, 12, 3, 1, 72, 576), ANYWHERE),     # few tiles
                                                           ((3, 100, 140, 12, 13, 3, 1, 78, 576), ANYWHERE),
                                                           ((3, 100, 100, 12, 13, 3, 1, 156, 576), ANYWHERE),
                                                           ((2, 192, 130, 9, 16, 3, 1, 144, 0), ANYWHERE),
                                                           ((2, 128, 64, 12, 12, 3, 1, 72, 576), ANYWHERE),      # few output channels
                                                           ((128, 256, 256, 28, 28, 3, 1, 8, 576), ANYWHERE),    # bands far below a tile
                                                           ((1, 64, 16, 7, 7, 3, 1, 1, 576), ANYWHERE),
                                                           ((128, 256, 256, 28, 28, 3, 1, 112, 64), GENERAL),    # blocks cut channels
                                                           ((2, 128, 200, 12, 12, 3, 2, 18, 576), GENERAL)]:     # stride 2
            stride = 2 if (pad == 2) else 1
            pad = 1 if stride == 2 else pad
            n = lib.ard_conv_workspace_bytes(D.BF16, N, Cc, H, W, Cout, k, k, stride, pad)
            ws = heap(n)
            big = N * max(Cc, Cout) * (H + 2) * (W + 2) * 4
            A, Wt, out, keep = (heap(big) for _ in range(4))
            D.launches(lib)
            before = D.last_bounds(lib)[0]
            rc = lib.ard_conv_fwd_blocks(D.BF16, N, Cc, H, W, Cout, k, k, stride, pad, x, y, A, Wt, keep, out, ws, n, None)
            assert rc == 0, lib.ard_last_error().decode()
            names = D.launches(lib)[1]
            assert [e for e in (PLAN, ANYWHERE, GENERAL) if e in names] == [engine], (N, Cc, Cout, x, y, names)
            if engine != GENERAL:   # (the plan rides in the copy's launch)
                assert "block_plan_kernel" not in names and "to_grid_src_kernel" in names, (H, W, names)
            if engine == PLAN:
                nb, six = D.last_bounds(lib)
                assert nb == 1 and 0 <= six[0] < six[1] <= six[2] and 0 <= six[3] < six[4] <= six[5]


def test_block_pattern_random_shapes_pass_the_proof():
    """Seeded random layers under the block pattern (forward, both gradient modes): whatever path dispatch picks,
    every LDS-direct launch passes the exhaustive bounds proof and every request is accepted or refused cleanly."""
    import random
    rnd = random.Random(52)
    with D.dry_run() as lib:
        heap = D.FakeHeap()
        fast = anywhere = 0
        for i in range(80):
            k = rnd.choice((1, 3, 3, 5))
            pad = rnd.choice((0, k // 2))
            H, W = rnd.randint(k + 4, 30), rnd.randint(k + 4, 30)
            N, Cc, Cout = rnd.randint(1, 6), rnd.choice((8, 40, 64, 100, 128, 192, 256)), rnd.choice((24, 65, 128, 130, 256, 300))
            if i >= 60:  # (enough images for 256 tiles)
                N = rnd.randint(100, 200)
            Ho, Wo = H + 2 * pad - k + 1, W + 2 * pad - k + 1
            x = rnd.choice((rnd.randint(1, Ho * Wo), max(1, Ho * Wo // rnd.randint(1, 8))))
            y = rnd.choice((0, 64 * k * k, 128 * k * k, k * k * rnd.randint(1, 70), rnd.randint(1, Cc * k * k)))
            n = lib.ard_conv_workspace_bytes(D.BF16, N, Cc, H, W, Cout, k, k, 1, pad)
            ws = heap(n)
            big = N * max(Cc, Cout) * (H + 2 * pad + 2) * (W + 2 * pad + 2) * 4
            A, Wt, dY, out, keep = (heap(big) for _ in range(5))
            D.launches(lib)
            rc = lib.ard_conv_fwd_blocks(D.BF16, N, Cc, H, W, Cout, k, k, 1, pad, x, y, A, Wt, keep, out, ws, n, None)
            assert rc == 0, (N, Cc, Cout, H, W, k, pad, x, y, lib.ard_last_error().decode())
            names = D.launches(lib)[1]
            fast += "gemm_direct_kernel" in names
            anywhere += "conv_block_fwd_kernel" in names
            for mode in (2, 3):
                rc = lib.ard_conv_bwd_blocks(mode, D.BF16, N, Cc, H, W, Cout, k, k, 1, pad, x, y, A, Wt, dY, keep, out, ws, n, None)
                assert rc == 0, (mode, N, Cc, Cout, H, W, k, pad, x, y, lib.ard_last_error().decode())
        assert fast >= 3 and anywhere >= 3, "the random shapes never reached the paths that skip dropped blocks"
        assert D.last_bounds(lib)[0] >= fast      # (reading them also resets the count for the next test)


def test_a_shortened_operand_is_rejected():
    """The proof is tight: with every operand pretended 8 elements shorter than it is, the dense 4096^3
    product (whose loaders read their operands to the last byte) must be refused, and nothing launched."""
    with D.dry_run() as lib:
        heap = D.FakeHeap()
        D.last_bounds(lib)
        _ok(lib, D.layer_calls(lib, heap, D.BF16, 4096, 4096, 4096, None, None, 0, ops=(0,)), "dense")
        n, six = D.last_bounds(lib)
        assert n == 1 and six[1] == six[2] and six[4] == six[5]      # both operands read up to their end
        D.launches(lib)
        lib.ard_debug_set_extent_slack(8)
        rc = D.layer_calls(lib, heap, D.BF16, 4096, 4096, 4096, None, None, 0, ops=(0,))
        assert rc == [-2] and "bounds proof" in lib.ard_last_error().decode()
        assert D.launches(lib)[0] == 0


def test_grouped_launch_of_a_dependency_level():
    """Independent calls recorded between ard_batch_begin and ard_batch_launch become one launch of the
    grouped kernel (plus one for their finishing passes); kernels the batch cannot hold are issued at once."""
    with D.dry_run() as lib:
        heap = D.FakeHeap()
        p1, p2 = (3, 2), (5, 1)
        assert lib.ard_batch_begin() == 0
        assert lib.ard_batch_begin() == -1            # already open
        _ok(lib, D.layer_calls(lib, heap, D.BF16, 1024, 2048, 2048, p2, p1, IN | OUT | WC, ops=(1, 2)), "level 4")
        assert D.launches(lib)[0] == 0                # everything recorded
        assert lib.ard_batch_launch(None) == 0
        n, names = D.launches(lib)
        assert names[0] == "group_kernel" and n <= 2, names
        assert lib.ard_batch_launch(None) == -1       # no batch open
        # the three products of the 10-neuron layer: one launch
        lib.ard_batch_begin()
        _ok(lib, D.layer_calls(lib, heap, D.BF16, 1024, 2048, 10, None, p2, IN | OUT), "level 3")
        assert lib.ard_batch_launch(None) == 0
        assert D.launches(lib) == (1, ["group_kernel"])
        # a call that gathers W itself issues the gather at once and records the product
        lib.ard_batch_begin()
        _ok(lib, D.layer_calls(lib, heap, D.BF16, 1024, 2048, 2048, p2, p1, IN | OUT, ops=(0,)), "gather inside")
        assert D.launches(lib) == (1, ["compact_weight_kernel"])
        assert lib.ard_batch_launch(None) == 0
        assert D.launches(lib) == (1, ["gemm_direct_kernel"])
        # fp32 is never recorded; abort drops a batch
        lib.ard_batch_begin()
        _ok(lib, D.layer_calls(lib, heap, D.F32, 64, 784, 1024, (2, 1), None, 0, ops=(0,)), "fp32")
        assert D.launches(lib)[0] >= 1
        lib.ard_batch_abort()
        assert lib.ard_batch_launch(None) == -1


@pytest.mark.parametrize("N,listed", [(328, True), (329, False)])
def test_pattern_gradients_of_layers_too_large_for_position_lists(N, listed):
    """64 channels of 224 x 224, 3 x 3: from 2^24 grid pixels (328.5 images) on the weight gradients of the row and block
    patterns leave the kernel that reads listed pixels for the one that reads them all; none is refused."""
    C, H, k, pad = 64, 224, 3, 1
    with D.dry_run() as lib:
        heap = D.FakeHeap()
        n = lib.ard_conv_workspace_bytes(D.BF16, N, C, H, H, C, k, k, 1, pad)
        ws, A, dY, Wt, out, keep = heap(n), heap(N * C * H * H * 2), heap(N * C * H * H * 2), heap(C * C * k * k * 2), heap(N * C * H * H * 2), heap(N * H * H)
        for mode in (6,):
            _ok(lib, [lib.ard_fmap_drop_conv(mode, D.BF16, N, C, H, H, C, k, k, 1, pad, 0.0, 0, A, Wt, dY, out, keep, None, None, None, ws, n, None)],
                f"rows {N} mode {mode}")
        for mode in (2, 3):
            D.launches(lib)
            _ok(lib, [lib.ard_conv_bwd_blocks(mode, D.BF16, N, C, H, H, C, k, k, 1, pad, 4 * H, 64 * k * k, A, Wt, dY, keep, out, ws, n, None)],
                f"blocks {N} mode {mode}")
            names = D.launches(lib)[1]
            if mode == 3:
                assert ("iota_kernel" in names) == (not listed), names   # (column block by column block, each with its own list of channels)
        D.last_bounds(lib)


@pytest.mark.parametrize("dtype", [D.F32, D.BF16])
def test_lstm_operands_beyond_one_launch(dtype):
    """A fused weight of 65532 x 316383: gathering it and scattering its gradient take several launches, and neither
    pass is refused (least of all after its other kernels have been enqueued)."""
    with D.dry_run() as lib:
        heap = D.FakeHeap()
        D.launches(lib)
        _ok(lib, D.lstm_calls(lib, heap, dtype, 2, 8, 300000, 16383, (2, 1)), "wide lstm")
        names = D.launches(lib)[1]
        assert names.count("lstm_prepare_kernel") == 4 and names.count("lstm_scatter_dw_kernel") == 3, names
        _ok(lib, D.lstm_calls(lib, heap, dtype, 3, 8, 30, 40, (2, 1)), "small lstm")
        names = D.launches(lib)[1]
        assert names.count("lstm_prepare_kernel") == 2 and names.count("lstm_scatter_dw_kernel") == 1, names
        D.last_bounds(lib)


def test_block_gradients_share_the_copy_of_dY_where_one_is_left():
    """The weight gradient takes the flag for any filter, and the copy itself where the data gradient left one that it can read: one
    column block or several, filters that keep the image's size and others."""
    with D.dry_run() as lib:
        heap = D.FakeHeap()
        for C, k, pad, x, y, shared in ((64, 3, 1, 50, 576, True), (64, 5, 2, 100, 0, True), (128, 3, 1, 40, 576, True), (64, 3, 0, 50, 576, False),
                                        (64, 3, 2, 50, 0, False), (128, 5, 0, 50, 1600, False), (24, 3, 1, 50, 72, False)):
            n = lib.ard_conv_workspace_bytes(D.BF16, 2, C, 40, 40, 8, k, k, 1, pad)
            ws, p = heap(n), heap(1 << 24)
            for mode in (2, 3 | 0x200):
                D.launches(lib)
                _ok(lib, [lib.ard_conv_bwd_blocks(mode, D.BF16, 2, C, 40, 40, 8, k, k, 1, pad, x, y, p, p, p, p, p, ws, n, None)], f"{C} {k} {pad} {mode}")
            assert (D.launches(lib)[1].count("to_grid_src_kernel") == 1) == shared, (C, k, pad, x, y)


def test_row_pattern_data_gradients_over_the_kept_positions():
    """Filters of several taps and more than 64 channels of dY; one tap has nothing to gain."""
    with D.dry_run() as lib:
        heap = D.FakeHeap()
        for (N, Cc, Cout, S, k), kept in [((128, 256, 256, 28, 3), True), ((128, 256, 256, 28, 1), False), ((63, 256, 80, 56, 1), False), ((128, 256, 64, 28, 3), False)]:
            n = lib.ard_conv_workspace_bytes(D.BF16, N, Cc, S, S, Cout, k, k, 1, k // 2)
            ws, p = heap(n), heap(1 << 20)
            D.launches(lib)
            _ok(lib, [lib.ard_fmap_drop_conv(5, D.BF16, N, Cc, S, S, Cout, k, k, 1, k // 2, 0.0, 0, None, p, p, p, p, None, None, None, ws, n, None)], "rows")
            assert ("conv_scatter_data_kernel" in D.launches(lib)[1]) == kept, (N, Cc, Cout, S, k)


def test_fp32_block_patterns_of_many_small_blocks_stay_in_one_pass():
    """A pass per column block where it is expected to be faster, else one over the patches of all."""
    with D.dry_run() as lib:
        heap = D.FakeHeap()
        for (N, Cc, Cout, S, k, cpb), passes in [((8, 64, 16, 16, 3, 64), 1), ((75, 64, 330, 16, 3, 32), 2), ((2, 48, 40, 14, 5, 3), 16),
                                                 ((2, 160, 16, 10, 5, 10), 16), ((2, 170, 16, 10, 5, 10), 0), ((36, 16, 2, 19, 1, 1), 0),
                                                 ((14, 32, 96, 28, 1, 2), 0), ((23, 8, 8, 13, 1, 1), 0), ((24, 128, 232, 28, 1, 128), 1)]:
            n = lib.ard_conv_workspace_bytes(D.F32, N, Cc, S, S, Cout, k, k, 1, k // 2)
            ws, p = heap(n), heap(1 << 20)
            D.launches(lib)
            _ok(lib, [lib.ard_conv_fwd_blocks(D.F32, N, Cc, S, S, Cout, k, k, 1, k // 2, S, cpb * k * k, p, p, p, p, ws, n, None)], "fp32 blocks")
            names = D.launches(lib)[1]
            assert names.count("add_bands_kernel") == passes and ("conv_gemm_kernel" in names) == (passes == 0), (N, Cc, Cout, S, k, cpb, names)


@pytest.mark.parametrize("dtype", [D.F32, D.BF16])
def test_lstm_workspace_holds_the_partial_sums_of_one_product(dtype):
    """Beside its operands a workspace has room for the largest product split 8 ways (at most 256 MiB) and, bf16, for what two
    more products can split into: 320 tiles of 64 x 64 each."""
    with D.dry_run() as lib:
        for T, B, I, H in ((64, 128, 1024, 1024), (35, 20, 1500, 1500), (8, 45, 56, 56), (64, 8, 4096, 2048), (100, 128, 64, 64)):
            es, Hp, Ip = 2 if dtype == D.BF16 else 4, -(-H // 8) * 8, -(-I // 8) * 8
            part = min(8 * 4 * 4 * Hp * max(Ip, Hp, B), 256 << 20)
            operands = es * (8 * Hp * (Ip + Hp) + 2 * T * B * Ip + T * (B + 31) * (Hp + 23)) + 16 * T * (B + 15) * (Hp + 23) + 4 * B * (Hp + H)
            more = 2 * 320 * 64 * 64 * 4 if dtype == D.BF16 else 0
            assert lib.ard_lstm_workspace_bytes(dtype, T, B, I, H, None) <= operands + part + more + (1 << 18), (T, B, I, H)


def test_lstm_shapes_reach_the_recurrences_their_gpu_tests_name():
    from test_gpu_lstm_staged import BEYOND_BWD, BEYOND_FWD
    with D.dry_run() as lib:
        heap = D.FakeHeap()
        for shapes, kernel in ((BEYOND_FWD, "lstm_persist_fwd_kernel"), (BEYOND_BWD, "lstm_persist_bwd_kernel")):
            for T, B, H in shapes:
                D.launches(lib)
                _ok(lib, D.lstm_calls(lib, heap, D.BF16, T, B, 16, H, (1, 1)), f"lstm {T} {B} {H}")
                assert kernel in D.launches(lib)[1], (kernel, T, B, H)
        D.last_bounds(lib)


def test_lstm_shapes_reach_every_recurrence_with_staging_wavefronts():
    from test_gpu_lstm_staged import STAGED
    with D.dry_run() as lib:
        heap = D.FakeHeap()
        reached = set()
        for (T, B, H), fwd, bwd in STAGED:
            D.launches(lib)
            _ok(lib, D.lstm_calls(lib, heap, D.BF16, T, B, 16, H, (1, 1)), f"lstm {T} {B} {H}")
            want = {f"lstm_staged_fwd_kernel {fwd[0]} {fwd[1]}"} | ({f"lstm_staged_bwd_kernel 2 {bwd}"} if bwd else set())
            got = {n for n in D.launches(lib)[1] if n.startswith("lstm_staged")}
            assert got == want, (got, T, B, H)
            reached |= got
        # every batch and width up to the end of the range: nothing else is launched, and the status word is there exactly
        # for the layers whose forward pass is one launch
        for B in (1, 16, 64, 65, 96, 112, 128, 129, 160, 200, 256, 300, 400, 512, 1100, 2100, 9000):
            for H in (8, 64, 128, 129, 200, 256, 257, 400, 512, 513, 600, 760, 768, 769, 1000, 1024, 1030, 1500):
                D.launches(lib)
                _ok(lib, D.lstm_calls(lib, heap, D.BF16, 2, B, 16, H, (1, 1)), f"lstm {B} {H}")
                names = D.launches(lib)[1]
                staged = {n for n in names if n.startswith("lstm_staged")}
                assert staged <= reached, (staged - reached, B, H)
                s, r = D.cpat((1, 1))
                one_launch = any(n.startswith(("lstm_xcd_fwd", "lstm_staged_fwd", "lstm_persist_fwd")) for n in names)
                assert (lib.ard_lstm_status_offset(D.BF16, 2, B, 16, H, r) != 2 ** 64 - 1) == one_launch, (names, B, H)
                assert any(n.startswith(("lstm_xcd_bwd", "lstm_staged_bwd", "lstm_persist_bwd")) for n in names) != ("lstm_cell_bwd_kernel" in names), (names, B, H)
        D.last_bounds(lib)


def test_lstm_shapes_reach_the_recurrences_with_a_block_per_xcd():
    from test_gpu_lstm_xcd import SHAPES
    with D.dry_run() as lib:
        heap = D.FakeHeap()
        for T, B, H, dp in SHAPES:
            D.launches(lib)
            _ok(lib, D.lstm_calls(lib, heap, D.BF16, T, B, 24, H, (dp, dp)), f"lstm {T} {B} {H}")
            names = D.launches(lib)[1]
            assert "lstm_xcd_fwd_kernel" in names and "lstm_xcd_bwd_kernel" in names, (names, T, B, H)
        D.last_bounds(lib)


def test_sensitivity_prediction_finds_its_bands_at_once():
    """How many bands a workgroup takes is worked out on each call: a layer of 18424 bands none of which leaves room for a
    second costs the host about what one of 98 bands costs (1.4 times; one number of bands after another, 50 times)."""
    import time
    with D.dry_run() as lib:
        heap = D.FakeHeap()

        def seconds(C, H, W, x):
            A, out = heap(2 * C * H * W * 4), [heap(1 << 24) for _ in range(3)]
            best = 1.0
            for _ in range(20):
                t = time.perf_counter()
                for _ in range(10):
                    _ok(lib, [lib.ard_sens_predict(D.F32, 2, C, H, W, 3, 3, 1, 1, x, 0, 300, 500, 0.5, 1, 0, A, *out, None)], "prediction")
                best = min(best, time.perf_counter() - t)
            assert "sens_predict_staged_kernel" in D.launches(lib)[1]
            return best
        small, large = seconds(256, 28, 28, 8), seconds(910, 188, 98, 1)
        assert large < 10 * small, (small, large)
