"""The calls of the extension _ardcall on tensors without memory behind them, in dry-run mode: what they accept, what
they refuse and how, without a GPU."""
import copy
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
