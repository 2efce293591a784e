"""Binding of libard.so: argument marshalling only.

Function names follow the C ABI (``include/ard.h``) without the ``ard_`` prefix.
Tensors are torch CUDA tensors used purely as device memory; every computation
runs in the library's HIP kernels.  The calls a training step issues come from the
extension ``_ardcall`` (``csrc/pyhost.cpp``), the others go through ctypes.  If the
library or the extension has not been built the first call raises -- there is no
fallback path.
"""
from __future__ import annotations

import copyreg
import ctypes as C
import os
from typing import Optional

import torch

HERE = os.path.dirname(os.path.abspath(__file__))
# (ARD_LIBRARY: another build of the same library, e.g. the host-sanitized one of build.py)
LIB_PATH = os.environ.get("ARD_LIBRARY") or os.path.join(HERE, "libard.so")

F32, BF16 = 0, 1
PAT_NONE, PAT_ROW, PAT_TILE, PAT_LIST = 0, 1, 2, 3
CONV_SELECT, CONV_FWD, CONV_BWD_DATA, CONV_BWD_WEIGHT, CONV_FWD_ROWS, CONV_BWD_DATA_ROWS, CONV_BWD_WEIGHT_ROWS = 0, 1, 2, 3, 4, 5, 6
CONV_REUSE_A, CONV_REUSE_DY = 0x100, 0x200
IN_COMPACT, OUT_COMPACT, W_COMPACT, DW_COMPACT = 1, 2, 4, 8


class ArdError(RuntimeError):
    def __init__(self, code: int, msg: str):
        super().__init__(f"libard error {code}: {msg}")
        self.code = code


class CPattern(C.Structure):
    _fields_ = [("kind", C.c_int32), ("dp", C.c_int32), ("b", C.c_int32),
                ("tile_r", C.c_int32), ("tile_c", C.c_int32), ("count", C.c_int32),
                ("d_keep", C.c_void_p), ("d_mask", C.c_void_p), ("d_rowptr", C.c_void_p),
                ("d_colptr", C.c_void_p), ("d_csc_rows", C.c_void_p)]


try:
    from . import _ardcall
except ImportError as e:   # not built: the names below are looked up in __getattr__, which says so
    _ardcall, _missing = None, e

if _ardcall is not None:
    _ardcall.configure(LIB_PATH, ArdError, torch._C._cuda_getCurrentRawStream)
    from ._ardcall import (batch, compact_weight, conv_bwd_blocks, conv_bwd_data, conv_bwd_rows, conv_bwd_weight,  # noqa: F401
                           conv_fwd, conv_fwd_blocks, conv_fwd_rows, conv_select, drop_gemm_bwd_data,
                           drop_gemm_bwd_weight, drop_gemm_bwd_weight_static, drop_gemm_fwd, lstm_bwd, lstm_fwd,
                           sens_block_pattern, sens_predict, sens_row_pattern)

    class Pattern(_ardcall.PatternBase):
        """Host description of a dropout pattern (keeps the tensors it points to alive):
        Pattern(kind, dp, b, tile_r, tile_c, keep, count, lists), or Pattern.row(dp, b),
        Pattern.tile(dp, b, tile_r, tile_c, lists=None), Pattern.list(keep, count=None)."""

        @staticmethod
        def list(keep: torch.Tensor, count=None):
            assert keep.dtype == torch.int32 and keep.is_cuda
            return Pattern(PAT_LIST, keep=keep, count=count)

        def c(self) -> CPattern:
            p = CPattern(self.kind, self.dp, self.b, self.tile_r, self.tile_c, self.count,
                         None, None, None, None, None)
            if self.kind == PAT_LIST and self.keep is not None:
                p.d_keep = self.keep.data_ptr()
            if self.kind == PAT_TILE and self.lists:
                p.d_keep = self.lists["keep"].data_ptr()
                p.d_mask = self.lists["mask"].data_ptr()
                p.d_rowptr = self.lists["rowptr"].data_ptr()
                p.d_colptr = self.lists["colptr"].data_ptr()
                p.d_csc_rows = self.lists["csc_rows"].data_ptr()
            return p

        # copies and pickles: the fields (which live in the base's C struct) and whatever else an instance was given
        _FIELDS = ("kind", "dp", "b", "tile_r", "tile_c", "keep", "count", "lists")

        def __reduce__(self):
            return copyreg.__newobj__, (type(self),), {**{f: getattr(self, f) for f in self._FIELDS}, **self.__dict__}

        def __setstate__(self, state):
            for name, value in state.items():
                setattr(self, name, value)


def __getattr__(name):
    if _ardcall is None and not name.startswith("_"):
        raise RuntimeError(f"the extension _ardcall is missing ({_missing}): build it with "
                           "`python -m paper_2203_05705_amd.build` (or __graft_entry__.build()); there is no fallback path")
    raise AttributeError(f"module {__name__!r} has no attribute {name!r}")


_lib = None

_SIGS = {
    "ard_search_k": (C.c_int32, [C.c_double, C.c_int32, C.c_uint64, C.c_void_p, C.c_void_p]),
    "ard_pattern_sample": (C.c_int32, [C.c_void_p, C.c_int32, C.c_uint64, C.c_uint64, C.c_uint32, C.c_void_p, C.c_void_p]),
    "ard_pattern_gen": (C.c_int32, [C.c_void_p, C.c_int32, C.c_int32] + [C.c_void_p] * 7),
    "ard_gemm_workspace_bytes": (C.c_size_t, [C.c_int32] * 4 + [C.c_void_p] * 2),
    "ard_compact_weight": (C.c_int32, [C.c_int32] * 3 + [C.c_void_p] * 5),
    "ard_drop_gemm_fwd": (C.c_int32, [C.c_int32] * 4 + [C.c_void_p] * 5 + [C.c_float, C.c_int32, C.c_int32, C.c_void_p, C.c_size_t, C.c_void_p]),
    "ard_drop_gemm_bwd_data": (C.c_int32, [C.c_int32] * 4 + [C.c_void_p] * 5 + [C.c_float, C.c_void_p, C.c_int32, C.c_void_p, C.c_size_t, C.c_void_p]),
    "ard_drop_gemm_bwd_weight": (C.c_int32, [C.c_int32] * 4 + [C.c_void_p] * 5 + [C.c_float, C.c_float, C.c_int32, C.c_void_p, C.c_size_t, C.c_void_p]),
    "ard_static_scratch_bytes": (C.c_size_t, []),
    "ard_drop_gemm_bwd_weight_static": (C.c_int32, [C.c_int32] * 4 + [C.c_void_p] * 5 + [C.c_float, C.c_float, C.c_int32, C.c_void_p]),
    "ard_batch_begin": (C.c_int32, []),
    "ard_batch_launch": (C.c_int32, [C.c_void_p]),
    "ard_batch_abort": (None, []),
    "ard_relu_bwd": (C.c_int32, [C.c_int32, C.c_int64] + [C.c_void_p] * 4),
    "ard_lstm_workspace_bytes": (C.c_size_t, [C.c_int32] * 5 + [C.c_void_p]),
    "ard_lstm_status_offset": (C.c_size_t, [C.c_int32] * 5 + [C.c_void_p]),
    "ard_lstm_fwd": (C.c_int32, [C.c_int32] * 5 + [C.c_void_p] * 7 + [C.c_size_t, C.c_void_p]),
    "ard_lstm_bwd": (C.c_int32, [C.c_int32] * 5 + [C.c_void_p] * 10 + [C.c_size_t, C.c_void_p]),
    "ard_conv_workspace_bytes": (C.c_size_t, [C.c_int32] * 10),
    "ard_fmap_drop_conv": (C.c_int32, [C.c_int32] * 11 + [C.c_double, C.c_int32] + [C.c_void_p] * 9 + [C.c_size_t, C.c_void_p]),
    "ard_conv_fwd_blocks": (C.c_int32, [C.c_int32] * 12 + [C.c_void_p] * 5 + [C.c_size_t, C.c_void_p]),
    "ard_conv_bwd_blocks": (C.c_int32, [C.c_int32] * 13 + [C.c_void_p] * 6 + [C.c_size_t, C.c_void_p]),
    "ard_sens_regions": (C.c_int32, [C.c_int32] * 10 + [C.c_void_p] * 3),
    "ard_sens_predict": (C.c_int32, [C.c_int32] * 13 + [C.c_float, C.c_uint64, C.c_uint64] + [C.c_void_p] * 5),
    "ard_sens_row_pattern": (C.c_int32, [C.c_int32] * 3 + [C.c_void_p, C.c_double, C.c_double, C.c_uint64, C.c_uint64] + [C.c_void_p] * 4),
    "ard_sens_block_pattern": (C.c_int32, [C.c_int32] * 3 + [C.c_void_p] * 3 + [C.c_int32, C.c_double, C.c_double, C.c_uint64, C.c_uint64] + [C.c_void_p] * 3),
    "ard_skew_normal_params": (C.c_int32, [C.c_double] * 3 + [C.c_void_p] * 2),
    "ard_skew_normal_pdf": (C.c_double, [C.c_double] * 4),
    "ard_prune_schedule": (C.c_int32, [C.c_int32] + [C.c_double] * 5 + [C.c_void_p]),
    "ard_kept_count": (C.c_int32, [C.c_void_p, C.c_int32]),
    "ard_compact_dim": (C.c_int32, [C.c_void_p, C.c_int32]),
    "ard_tile_grid": (C.c_int32, [C.c_void_p, C.c_int32, C.c_int32, C.c_void_p, C.c_void_p]),
    "ard_conv_out_size": (C.c_int32, [C.c_int32] * 4),
    "ard_debug_set_dry_run": (None, [C.c_int32]),
    "ard_debug_dry_launches": (C.c_int32, [C.c_char_p, C.c_size_t]),
    "ard_debug_dry_instances": (C.c_int32, [C.c_char_p, C.c_size_t]),
    "ard_debug_last_bounds": (C.c_int32, [C.c_void_p]),
    "ard_debug_compared_slabs": (C.c_int64, []),
    "ard_debug_set_extent_slack": (None, [C.c_int64]),
    "ard_last_error": (C.c_char_p, []),
    "ard_version": (C.c_int32, []),
}


def exported_symbols():
    """Names every build of the library must export (mirrors include/ard.h)."""
    return sorted(_SIGS)


def lib():
    """The loaded library; raises if it has not been built (no fallback exists)."""
    global _lib
    if _lib is None:
        if not os.path.exists(LIB_PATH):
            raise RuntimeError(f"{LIB_PATH} is missing: build it with `python -m paper_2203_05705_amd.build` "
                               "(or __graft_entry__.build()); there is no fallback path")
        handle = C.CDLL(LIB_PATH)
        for name, (res, args) in _SIGS.items():
            fn = getattr(handle, name)
            fn.restype, fn.argtypes = res, args
        _lib = handle
    return _lib


def _check(code: int):
    if code != 0:
        raise ArdError(code, lib().ard_last_error().decode())


def _dtype_code(t: torch.Tensor) -> int:
    if t.dtype == torch.float32:
        return F32
    if t.dtype == torch.bfloat16:
        return BF16
    raise TypeError(f"unsupported dtype {t.dtype}")


def _stream(stream):
    return (torch.cuda.current_stream() if stream is None else stream).cuda_stream


def _pref(p: "Optional[Pattern]"):
    if p is None:
        return None, None
    cp = p.c()
    return cp, C.byref(cp)


def _ptr(t: Optional[torch.Tensor]):
    return None if t is None else t.data_ptr()


_ALLOC = torch.empty


def set_output_allocator(fn=None):
    """Every output tensor the wrappers below create comes from fn(shape, dtype=..., device=...)
    (default torch.empty).  Tests install an allocator that poisons outputs and fences them with
    guard bands; returns the previous allocator."""
    global _ALLOC
    prev, _ALLOC = _ALLOC, (torch.empty if fn is None else fn)
    _ardcall.set_allocator(None if _ALLOC is torch.empty else _ALLOC)
    return prev


def _out(shape, dtype, device):
    return _ALLOC(tuple(int(v) for v in shape), dtype=dtype, device=device)


def _dev(t: torch.Tensor):
    assert t.is_cuda and t.is_contiguous(), "device-resident contiguous tensors only"
    return t


def to_device(a, device="cuda") -> torch.Tensor:
    """Host array -> device tensor with the bytes unchanged: uint16 arrays are bf16 bit
    patterns, float32 stays float32, integer arrays keep their type."""
    import numpy as np
    a = np.ascontiguousarray(a)
    if a.dtype == np.uint16:
        return torch.from_numpy(a.view(np.int16).copy()).to(device).view(torch.bfloat16)
    return torch.from_numpy(a.copy()).to(device)


# ---- host-side pattern distribution and sampling -----------------------------

def search_k(p: float, n: int, seed: int = 0):
    """Returns (k: list[float], cdf: list[int]) from the library's host search."""
    k = (C.c_double * n)()
    cdf = (C.c_uint64 * n)()
    _check(lib().ard_search_k(p, n, seed, k, cdf))
    return list(k), list(cdf)


def pattern_sample(cdf, seed: int, it: int, stream_id: int):
    arr = (C.c_uint64 * len(cdf))(*[int(c) for c in cdf])
    dp, b = C.c_int32(), C.c_int32()
    _check(lib().ard_pattern_sample(arr, len(cdf), seed, it, stream_id, C.byref(dp), C.byref(b)))
    return dp.value, b.value


def prune_schedule(n_epochs: int, total: float, mean: float, var: float, lam: float, p_max: float = 1.0):
    """Per-epoch prune possibilities along the skew-normal curve of Section 5.3 (host doubles)."""
    out = (C.c_double * n_epochs)()
    _check(lib().ard_prune_schedule(n_epochs, total, mean, var, lam, p_max, out))
    return list(out)


# ---- device entry points ---------------------------------------------------------

def pattern_gen(pat: "Pattern", rows: int, cols: int = 0, device="cuda", stream=None) -> dict:
    """Mask, kept list, count (and tile offsets) as device tensors."""
    cp, ref = _pref(pat)
    if pat.kind == PAT_TILE:
        tr, tc = C.c_int32(), C.c_int32()
        _check(lib().ard_tile_grid(ref, rows, cols, C.byref(tr), C.byref(tc)))
        TR, TC = tr.value, tc.value
        n = TR * TC
        out = dict(mask=_out((n,), torch.uint8, device),
                   keep=torch.full((n,), -1, dtype=torch.int32, device=device),
                   count=torch.zeros(1, dtype=torch.int32, device=device),
                   rowptr=_out((TR + 1,), torch.int32, device),
                   colptr=_out((TC + 1,), torch.int32, device),
                   csc_rows=torch.full((n,), -1, dtype=torch.int32, device=device))
        _check(lib().ard_pattern_gen(ref, rows, cols, out["mask"].data_ptr(), out["keep"].data_ptr(),
                                     out["count"].data_ptr(), out["rowptr"].data_ptr(), out["colptr"].data_ptr(),
                                     out["csc_rows"].data_ptr(), _stream(stream)))
        return out
    n = max(rows, 1)
    out = dict(mask=_out((n,), torch.uint8, device),
               keep=torch.full((n,), -1, dtype=torch.int32, device=device),
               count=torch.zeros(1, dtype=torch.int32, device=device))
    _check(lib().ard_pattern_gen(ref, rows, cols, out["mask"].data_ptr(), out["keep"].data_ptr(),
                                 out["count"].data_ptr(), None, None, None, _stream(stream)))
    return out


def gemm_workspace_bytes(dtype_code, B, I, O, pat_out=None, pat_in=None) -> int:
    _, ro = _pref(pat_out)
    _, ri = _pref(pat_in)
    return int(lib().ard_gemm_workspace_bytes(dtype_code, B, I, O, ro, ri))


def _workspace(nbytes: int, device, ws: Optional[torch.Tensor]):
    if ws is not None:
        return ws
    return torch.empty(max(nbytes, 1), dtype=torch.uint8, device=device)


def kept_count(pat: "Optional[Pattern]", units: int) -> int:
    """Number of kept units of a ROW / LIST / NONE pattern over `units` (asked of the library)."""
    _, r = _pref(pat)
    n = lib().ard_kept_count(r, units)
    if n < 0:
        _check(n)
    return n


def pad8(n: int) -> int:
    """Stored extent of a compact axis with n kept units (asked of the library)."""
    return lib().ard_compact_dim(None, n)


def pad_compact(t: torch.Tensor) -> torch.Tensor:
    """[B, count] -> [B, pad8(count)] with zero padding: the compact activation layout."""
    B, n = t.shape
    out = torch.zeros((B, pad8(n)), dtype=t.dtype, device=t.device)
    out[:, :n] = t
    return out


def relu_bwd(dY, Y, out=None, stream=None):
    _dev(dY), _dev(Y)
    dX = _out(dY.shape, dY.dtype, dY.device) if out is None else out
    _check(lib().ard_relu_bwd(_dtype_code(dY), dY.numel(), dY.data_ptr(), Y.data_ptr(), dX.data_ptr(), _stream(stream)))
    return dX


# ---- LSTM -------------------------------------------------------------------------------

def lstm_workspace_bytes(dtype_code, T, B, I, H, pat=None) -> int:
    _, r = _pref(pat)
    return int(lib().ard_lstm_workspace_bytes(dtype_code, T, B, I, H, r))


def lstm_status_offset(dtype_code, T, B, I, H, pat=None):
    """Byte offset in the workspace of the recurrence's give-up flag, or None (launch-per-step path)."""
    _, r = _pref(pat)
    off = int(lib().ard_lstm_status_offset(dtype_code, T, B, I, H, r))
    return None if off == (1 << 64) - 1 else off


# ---- convolution with dropped input feature maps ---------------------------------------------

def conv_workspace_bytes(dtype_code, N, C, H, W, Cout, kh, kw, stride, pad) -> int:
    return int(lib().ard_conv_workspace_bytes(dtype_code, N, C, H, W, Cout, kh, kw, stride, pad))


def fmap_drop_conv(mode, shape, dtype_code, Cout, ksize, stride, pad, rate=0.0, n_keep=0, A=None, Wt=None, dY=None,
                   out=None, mask=None, keep=None, count=None, score=None, ws=None, stream=None):
    """Raw call of ard_fmap_drop_conv; `shape` = (N, C, H, W) of the activations."""
    N, Cc, H, W = shape
    kh, kw = ksize
    dev = next(t.device for t in (A, Wt, dY, out, keep) if t is not None)
    ws = _workspace(conv_workspace_bytes(dtype_code, N, Cc, H, W, Cout, kh, kw, stride, pad), dev, ws)
    _check(lib().ard_fmap_drop_conv(mode, dtype_code, N, Cc, H, W, Cout, kh, kw, stride, pad, float(rate), int(n_keep),
                                    _ptr(A), _ptr(Wt), _ptr(dY), _ptr(out), _ptr(mask), _ptr(keep), _ptr(count),
                                    _ptr(score), ws.data_ptr(), ws.numel(), _stream(stream)))


def sens_regions(shape, ksize, stride, pad, x, y=0):
    """(rows, row_bands, col_blocks) of the input matrix of one image under x-by-y regions."""
    N, Cc, H, W = shape
    r, rb, cb = C.c_int32(), C.c_int32(), C.c_int32()
    _check(lib().ard_sens_regions(N, Cc, H, W, ksize[0], ksize[1], stride, pad, x, y, C.byref(r), C.byref(rb), C.byref(cb)))
    return r.value, rb.value, cb.value
