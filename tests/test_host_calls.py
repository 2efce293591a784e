"""The calls of the extension _ardcall on tensors without memory behind them, in dry-run mode: what they accept, what
they refuse and how, without a GPU."""
import copy
import inspect
import os
import pickle
import subprocess
import sys
import textwrap
from types import SimpleNamespace

import pytest
import torch

from dryrun import FakeHeap, dry_run
from paper_2203_05705_amd import binding as ard

STREAM = SimpleNamespace(cuda_stream=0)   # (torch has no current stream without a GPU)
_heap = FakeHeap()


def fake(*shape, dtype=torch.float32):
    """A contiguous CUDA tensor at an address nothing is mapped at."""
    meta = torch.empty(shape, dtype=dtype, device="meta")
    n = max(meta.numel(), 1) * dtype.itemsize
    storage = torch._C._construct_storage_from_data_pointer(_heap(n), torch.device("cuda:0"), n)
    return torch._C._construct_CUDA_Tensor_From_Storage_And_Metadata(
        dict(dtype=dtype, size=meta.shape, stride=meta.stride(), storage_offset=0, device=torch.device("cuda:0"), data_ptr=0, nbytes=n), storage)


def fake_ws(n=1 << 26):
    return fake(n, dtype=torch.uint8)


# Every entry point that takes addresses, as a function of its first tensor (the others exist): a tensor without
# storage in that place (vmap's) raises as its data_ptr() does.
def _entry_points():
    X, W, Y, ws = fake(64, 128), fake(256, 128), fake(64, 256), fake_ws()
    x, Wl, hl, c, g = fake(3, 8, 32), fake(128, 64), fake(3, 8, 32), fake(3, 8, 32), fake(3, 8, 128)
    A, Wt, Yc, keep = fake(2, 8, 6, 6), fake(4, 8, 3, 3), fake(2, 4, 6, 6), fake(8, dtype=torch.int32)
    u8, i32 = fake(72, dtype=torch.uint8), fake(72, dtype=torch.int32)
    rows = dict(mask=u8, keep=i32)
    sel = dict(mask=u8, keep=keep, count=i32, score=fake(8, dtype=torch.int64))
    kw = dict(ws=ws, stream=STREAM)
    return dict(
        compact_weight=(W, lambda t: ard.compact_weight(t, out=Y, stream=STREAM)),
        drop_gemm_fwd=(X, lambda t: ard.drop_gemm_fwd(t, W, out=Y, **kw)),
        drop_gemm_bwd_data=(Y, lambda t: ard.drop_gemm_bwd_data(t, W, out=X, **kw)),
        drop_gemm_bwd_weight=(Y, lambda t: ard.drop_gemm_bwd_weight(t, X, out=W, **kw)),
        drop_gemm_bwd_weight_static=(Y, lambda t: ard.drop_gemm_bwd_weight_static(t, X, None, None, W, stream=STREAM)),
        lstm_fwd=(x, lambda t: ard.lstm_fwd(t, Wl, out=(hl, c, g), **kw)),
        lstm_bwd=(x, lambda t: ard.lstm_bwd(t, Wl, None, hl, c, g, hl, out=(x, Wl), **kw)),
        conv_select=(A, lambda t: ard.conv_select(t, 0.5, out=sel, **kw)),
        conv_fwd=(A, lambda t: ard.conv_fwd(t, Wt, keep, 4, out=Yc, **kw)),
        conv_bwd_data=(Yc, lambda t: ard.conv_bwd_data(t, Wt, keep, 4, (6, 6), out=A, **kw)),
        conv_bwd_weight=(Yc, lambda t: ard.conv_bwd_weight(t, A, keep, 4, out=Wt, **kw)),
        conv_fwd_rows=(A, lambda t: ard.conv_fwd_rows(t, Wt, rows, 4, out=Yc, **kw)),
        conv_bwd_rows=(Yc, lambda t: ard.conv_bwd_rows(t, A, Wt, rows, out=(A, Wt), **kw)),
        conv_fwd_blocks=(A, lambda t: ard.conv_fwd_blocks(t, Wt, u8, 12, 0, out=Yc, **kw)),
        conv_bwd_blocks=(Yc, lambda t: ard.conv_bwd_blocks(t, A, Wt, u8, 12, 0, out=(A, Wt), **kw)),
        sens_predict=(A, lambda t: ard.sens_predict(t, (3, 3), 1, 1, 12, 0, 300, 500, 0.5, 1, 0, stream=STREAM)))


@pytest.mark.parametrize("name", ["compact_weight", "drop_gemm_fwd", "drop_gemm_bwd_data", "drop_gemm_bwd_weight", "drop_gemm_bwd_weight_static",
                                  "lstm_fwd", "lstm_bwd", "conv_select", "conv_fwd", "conv_bwd_data", "conv_bwd_weight", "conv_fwd_rows",
                                  "conv_bwd_rows", "conv_fwd_blocks", "conv_bwd_blocks", "sens_predict"])
def test_an_argument_without_storage_raises(name):
    """In a process of its own: raised where the interpreter lock had been given up, it ended the interpreter."""
    code = f"""
        import torch
        import test_host_calls as T
        T.ard.set_output_allocator(lambda shape, dtype, device: T.fake(*shape, dtype=dtype))
        with T.dry_run():
            first, call = T._entry_points()[{name!r}]
            call(first)
            batched = T.fake(2, *first.shape, dtype=first.dtype)
            try:
                torch.vmap(call)(batched)
            except RuntimeError as e:
                assert "storage" in str(e), e
                print("raised")
            call(first)
    """
    here = os.path.dirname(os.path.abspath(__file__))
    r = subprocess.run([sys.executable, "-c", textwrap.dedent(code)], cwd=os.path.dirname(here), capture_output=True, text=True, timeout=300,
                       env=dict(os.environ, PYTHONPATH=os.pathsep.join((here, os.path.dirname(here)))))
    assert r.returncode == 0 and "raised" in r.stdout, (r.returncode, r.stdout, r.stderr[-2000:])


class _Named(ard.Pattern):
    """A program's own kind of pattern."""


@pytest.mark.parametrize("copier", [copy.copy, copy.deepcopy] + [lambda p, v=v: pickle.loads(pickle.dumps(p, v)) for v in range(6)])
def test_patterns_and_batches_can_be_copied_and_pickled(copier):
    keep = torch.tensor([1, 4, 6], dtype=torch.int32)
    named = _Named(ard.PAT_ROW, 4, 2)
    named.label = "fc1"
    for p in (ard.Pattern(), ard.Pattern.row(3, 2), ard.Pattern.tile(2, 1, 32, 64, lists=dict(keep=keep)), ard.Pattern(ard.PAT_LIST, keep=keep),
              ard.Pattern(ard.PAT_LIST, keep=keep, count=2), named):
        q = copier(p)
        assert type(q) is type(p) and q is not p
        for f in ("kind", "dp", "b", "tile_r", "tile_c", "count"):
            assert getattr(q, f) == getattr(p, f), f
        assert (q.keep is None) == (p.keep is None) and (p.keep is None or torch.equal(q.keep, p.keep))
        assert (q.lists is None) == (p.lists is None) and (p.lists is None or torch.equal(q.lists["keep"], keep))
        assert (q.keep is p.keep) == (copier is copy.copy or p.keep is None)
    assert copier(named).label == "fc1"
    assert copier(ard.batch()).stream is None


def test_constructors_called_through_a_derived_class_give_a_plain_pattern():
    class Layer(ard.Pattern):
        def __new__(cls, name):
            return super().__new__(cls)

        def __init__(self, name):
            super().__init__(ard.PAT_ROW, 2, 1)
    for p in (Layer.row(3, 2), Layer.tile(3, 2, 8, 8)):
        assert type(p) is ard.Pattern and (p.dp, p.b) == (3, 2)
    assert Layer("fc1").dp == 2


def test_activations_of_more_than_two_dimensions_are_flattened():
    """B is the first dimension; the weight (or I and O) says how much follows."""
    X, W, Y, ws = fake(64, 2, 8, 8), fake(256, 128), fake(64, 256), fake_ws()
    kw = dict(ws=ws, stream=STREAM)
    with dry_run():
        assert ard.drop_gemm_fwd(X, W, out=Y, **kw) is Y
        assert ard.drop_gemm_bwd_data(fake(64, 16, 16), W, out=X, **kw) is X
        assert ard.drop_gemm_bwd_weight(fake(64, 16, 16), X, out=W, I=128, O=256, **kw) is W
        assert ard.drop_gemm_bwd_weight_static(Y, X, None, None, W, I=128, stream=STREAM) is W
        W4 = fake(256, 2, 8, 8)
        assert ard.drop_gemm_fwd(X, W4, out=Y, I=128, O=256, **kw) is Y
        p = ard.Pattern.row(2, 1)
        ard.drop_gemm_fwd(fake(64, 64, 1), W, None, p, flags=ard.IN_COMPACT, out=Y, **kw)
        # a convolution's gradient: the first two dimensions count
        A, dA = fake(2, 8, 6, 6), fake(2, 8, 6, 6)
        ard.conv_bwd_weight(fake(2, 4, 36), A, None, 8, out=fake(4, 8, 3, 3), **kw)
        ard.conv_bwd_data(fake(2, 4, 36), fake(4, 8, 3, 3), None, 8, None, out=dA, **kw)   # (sizes come from `out`)
        x, h, c, g = fake(3, 8, 32), fake(3, 8, 32), fake(3, 8, 32), fake(3, 8, 128)
        ard.lstm_bwd(x, fake(128, 8, 8), None, h, c, g, h, out=(x, fake(128, 64)), **kw)


def test_counts_and_rates_are_taken_from_what_int_and_float_take():
    A, Wt, Y, ws = fake(2, 8, 6, 6), fake(4, 8, 3, 3), fake(2, 4, 6, 6), fake_ws()
    keep, u8 = fake(72, dtype=torch.int32), fake(72, dtype=torch.uint8)
    kw = dict(ws=ws, stream=STREAM)
    with dry_run():
        for four in (4, 4.0, "4", torch.tensor(4), torch.tensor(4.0), True + 3):
            ard.conv_fwd(A, Wt, keep, four, out=Y, **kw)
            ard.conv_bwd_data(Y, Wt, keep, four, (6, 6), out=A, **kw)
            ard.conv_bwd_weight(Y, A, keep, four, out=Wt, **kw)
            ard.conv_fwd_rows(A, Wt, dict(keep=keep, mask=u8), four, out=Y, **kw)
            ard.conv_fwd_blocks(A, Wt, u8, four, 72.0, out=Y, **kw)
            ard.conv_bwd_blocks(Y, A, Wt, u8, four, "72", out=(A, Wt), **kw)
        for half in (0.5, "0.5", torch.tensor(0.5)):
            ard.conv_select(A, half, out=dict(mask=u8, keep=keep, count=None, score=None), **kw)
            ard.drop_gemm_fwd(fake(16, 8), fake(8, 8), alpha=half, out=fake(16, 8), **kw)
        ard.conv_fwd_rows(A, Wt, dict(keep=None, mask=u8), 0, out=Y, **kw)   # (an empty list needs no address)
        with pytest.raises((TypeError, ValueError)):
            ard.conv_fwd(A, Wt, keep, "four", out=Y, **kw)
        with pytest.raises(TypeError):
            ard.conv_fwd(A, Wt, keep, None, out=Y, **kw)


def test_what_was_refused_stays_refused():
    X, W, Y, ws = fake(64, 128), fake(256, 128), fake(64, 256), fake_ws()
    A, Wt, keep = fake(2, 8, 6, 6), fake(4, 8, 3, 3), fake(8, dtype=torch.int32)
    sel = dict(mask=fake(8, dtype=torch.uint8), keep=keep, count=keep, score=fake(8, dtype=torch.int64))
    kw = dict(ws=ws, stream=STREAM)
    with dry_run():
        for error, call in [
                (ValueError, lambda: ard.compact_weight(fake(4, 4, 4), out=W, stream=STREAM)),
                (AssertionError, lambda: ard.drop_gemm_fwd(X.t(), W, out=Y, **kw)),
                (IndexError, lambda: ard.drop_gemm_fwd(X, fake(256), out=Y, **kw)),
                (IndexError, lambda: ard.drop_gemm_bwd_weight(fake(64), X, out=W, **kw)),
                (IndexError, lambda: ard.drop_gemm_fwd(fake(64), W, None, None, flags=ard.IN_COMPACT, out=Y, **kw)),
                (ValueError, lambda: ard.drop_gemm_fwd(X, W, None, ard.Pattern.row(2, 1), flags=ard.IN_COMPACT, out=Y, **kw)),
                (TypeError, lambda: ard.drop_gemm_fwd(X, W, out=Y, I=128.0, **kw)),
                (AssertionError, lambda: ard.drop_gemm_fwd(X, W, flags=ard.W_COMPACT, out=Y, **kw)),
                (ValueError, lambda: ard.lstm_fwd(X, W, out=(X, X, X), **kw)),
                (AssertionError, lambda: ard.lstm_fwd(fake(3, 8, 32), fake(128, 8, 8), out=(X, X, X), **kw)),
                (ValueError, lambda: ard.conv_fwd(A, fake(4, 8, 9), keep, 4, out=A, **kw)),
                (ValueError, lambda: ard.conv_select(A, 0.5, ksize=(3, 3, 3), out=sel, **kw)),
                (ValueError, lambda: ard.conv_bwd_weight(A, A, keep, 4, ksize=(3,), out=Wt, **kw)),
                (TypeError, lambda: ard.conv_bwd_weight(A, A, keep, 4, ksize=(3.0, 3.0), out=Wt, **kw)),
                (TypeError, lambda: ard.conv_fwd(A, Wt, keep, 4, stride=1.0, out=A, **kw)),
                (ard.ArdError, lambda: ard.conv_fwd_rows(A, Wt, dict(keep=None, mask=None), 4, out=A, **kw))]:
            with pytest.raises(error):
                call()


def test_errors_of_torch_keep_their_types():
    """The workspace a call makes itself: where torch refuses it, the error is the one torch.empty raises."""
    X, W, Y = fake(64, 128, dtype=torch.bfloat16), fake(256, 128, dtype=torch.bfloat16), fake(64, 256, dtype=torch.bfloat16)

    class Refuse(torch.utils._python_dispatch.TorchDispatchMode):
        def __torch_dispatch__(self, func, types, args=(), kwargs=None):
            raise torch.OutOfMemoryError("no room")
    with dry_run(), Refuse(), pytest.raises(torch.OutOfMemoryError, match="no room"):
        ard.drop_gemm_fwd(X, W, out=Y, stream=STREAM)


def test_signatures_can_be_read():
    """What help(), editors and wrappers that look at a function's parameters see."""
    gemm = "pat_out=None, pat_in=None, alpha=1.0, {}flags=0, out=None, ws=None, stream=None, I=None, O=None"
    conv = "stride=1, pad=1, ws=None, stream=None, out=None"
    want = dict(
        compact_weight="W, pat_out=None, pat_in=None, out=None, stream=None", drop_gemm_fwd="X, W, " + gemm.format("relu=False, "),
        drop_gemm_bwd_data="dY, W, " + gemm.format("relu_src=None, "), drop_gemm_bwd_weight="dY, X, " + gemm.format("beta=0.0, "),
        drop_gemm_bwd_weight_static="dY, X, pat_out, pat_in, out, alpha=1.0, beta=0.0, flags=0, stream=None, I=None, O=None",
        lstm_fwd="x, W, pat=None, ws=None, stream=None, out=None", lstm_bwd="x, W, pat, h, c, gates, dh, ws=None, stream=None, out=None",
        conv_select="A, rate, Cout=1, ksize=(3, 3), " + conv, conv_fwd="A, Wt, keep, n_keep, " + conv + ", reuse=0",
        conv_bwd_data="dY, Wt, keep, n_keep, in_hw, " + conv + ", reuse=0",
        conv_bwd_weight="dY, A, keep, n_keep, ksize=(3, 3), " + conv + ", reuse=0", conv_fwd_rows="A, Wt, row_pat, n_keep, " + conv,
        conv_bwd_rows="dY, A, Wt, row_pat, " + conv + ", reuse=0", conv_fwd_blocks="A, Wt, block_keep, x, y, " + conv,
        conv_bwd_blocks="dY, A, Wt, block_keep, x, y, " + conv,
        sens_predict="A, ksize, stride, pad, x, y, k_permille, t_permille, threshold, seed, iteration, stream=None",
        sens_row_pattern="sens, rows, x, m, n, seed, iteration, stream=None", sens_block_pattern="pred, balance, m, n, seed, iteration, stream=None",
        batch="stream=None", Pattern="kind=0, dp=1, b=1, tile_r=0, tile_c=0, keep=None, count=None, lists=None")
    for name, params in want.items():
        assert str(inspect.signature(getattr(ard, name))) == f"({params})", name
    assert str(inspect.signature(ard.Pattern.row)) == "(dp, b)"
    assert str(inspect.signature(ard.Pattern.tile)) == "(dp, b, tile_r, tile_c, lists=None)"
