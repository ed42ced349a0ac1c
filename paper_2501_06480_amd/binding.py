"""Python binding of the C-ABI library declared in ``include/fwa.h``.

Argument marshalling only: every step of the attention path runs in the HIP
kernels of ``libfwa.so``.  torch supplies device memory and the stream.  The
marshalling of the tensor calls is native (``csrc/torch_binding.cpp``, built as
``_fwa_torch``); the queries and the call that allocates nothing go through
ctypes.  There is no CPU fallback: when the libraries have not been built, or a
call is made without a GPU tensor, an exception is raised.
"""
from __future__ import annotations

import ctypes
import os
from typing import Optional

FWA_F32 = 0
FWA_BF16 = 1
FWA_F16 = 2

FWA_OK = 0
FWA_ERR_NULL = 1
FWA_ERR_SHAPE = 2
FWA_ERR_UNSUPPORTED = 3
FWA_ERR_ALIGN = 4
FWA_ERR_WORKSPACE = 5
FWA_ERR_LAUNCH = 6
FWA_ERR_ALIAS = 7
FWA_NOALLOC_SCRATCH_BYTES = 16 * 1024 * 1024

_HERE = os.path.dirname(os.path.abspath(__file__))
_LIB_PATH = os.path.join(_HERE, "libfwa.so")
_lib = None

EXPORTS = ("fwa_forward", "fwa_forward_strided", "fwa_forward_labels", "fwa_backward", "fwa_backward_strided",
           "fwa_backward_labels", "fwa_backward_noalloc",
           "fwa_backward_workspace_bytes", "fwa_bias_gather", "fwa_bias_scatter", "fwa_status_string")


class FwaError(RuntimeError):
    def __init__(self, code: int, what: str):
        super().__init__(f"{what}: {fwa_status_string(code)} (code {code})")
        self.code = code


def library_path() -> str:
    return _LIB_PATH


def native_path() -> str:
    """The native marshalling module beside the library."""
    return os.path.join(_HERE, "_fwa_torch.so")


def load_library():
    """Load ``libfwa.so`` (built in-tree by ``paper_2501_06480_amd.build``)."""
    global _lib
    if _lib is not None:
        return _lib
    if not os.path.exists(_LIB_PATH):
        raise RuntimeError(
            f"{_LIB_PATH} is missing: build it with `python -m paper_2501_06480_amd.build` "
            "(hipcc, gfx950). There is no fallback path.")
    lib = ctypes.CDLL(_LIB_PATH)
    vp, i64, ci, cf, sz = ctypes.c_void_p, ctypes.c_int64, ctypes.c_int, ctypes.c_float, ctypes.c_size_t
    lib.fwa_forward.restype = ci
    lib.fwa_forward.argtypes = [vp, vp, vp, vp, i64, ci, ci, ci, cf, vp, vp, ci, ci, vp]
    lib.fwa_forward_strided.restype = ci
    lib.fwa_forward_strided.argtypes = [vp, vp, vp, vp, i64, ci, ci, ci, cf, i64, i64, vp, vp, ci, ci, vp]
    lib.fwa_forward_labels.restype = ci
    lib.fwa_forward_labels.argtypes = [vp, vp, vp, vp, i64, ci, ci, ci, cf, i64, i64, vp, ci, vp, cf, ci, ci, vp]
    lib.fwa_backward_labels.restype = ci
    lib.fwa_backward_labels.argtypes = [vp, vp, vp, vp, vp, vp, vp, vp, i64, ci, ci, ci, cf, i64, i64, i64,
                                        vp, ci, vp, cf, ci, ci, vp, sz, vp]
    lib.fwa_backward.restype = ci
    lib.fwa_backward.argtypes = [vp, vp, vp, vp, vp, vp, vp, vp, i64, ci, ci, ci, cf, vp, vp, ci, ci,
                                 vp, sz, vp]
    lib.fwa_backward_noalloc.restype = ci
    lib.fwa_backward_noalloc.argtypes = [vp, vp, vp, vp, vp, vp, vp, vp, i64, ci, ci, ci, cf, vp, vp, ci, ci, vp]
    lib.fwa_backward_strided.restype = ci
    lib.fwa_backward_strided.argtypes = [vp, vp, vp, vp, vp, vp, vp, vp, i64, ci, ci, ci, cf, i64, i64, i64,
                                         vp, vp, ci, ci, vp, sz, vp]
    lib.fwa_backward_workspace_bytes.restype = sz
    lib.fwa_backward_workspace_bytes.argtypes = [i64, ci, ci, ci, ci, ci]
    lib.fwa_bias_gather.restype = ci
    lib.fwa_bias_gather.argtypes = [vp, vp, ci, ci, vp]
    lib.fwa_bias_scatter.restype = ci
    lib.fwa_bias_scatter.argtypes = [vp, vp, ci, ci, vp]
    lib.fwa_status_string.restype = ctypes.c_char_p
    lib.fwa_status_string.argtypes = [ci]
    _lib = lib
    return lib


def fwa_status_string(code: int) -> str:
    return load_library().fwa_status_string(int(code)).decode()


def _dtype_code(t) -> int:
    torch = _torch()
    if t.dtype == torch.float32:
        return FWA_F32
    if t.dtype == torch.bfloat16:
        return FWA_BF16
    if t.dtype == torch.float16:
        return FWA_F16
    raise TypeError(f"unsupported tensor dtype {t.dtype}")


def _dev_ptr(t, name: str, like=None, f32: bool = False) -> Optional[int]:
    if t is None:
        return None
    if not getattr(t, "is_cuda", False):
        raise TypeError(f"{name} must be a GPU tensor (there is no CPU path)")
    if not t.is_contiguous():
        raise ValueError(f"{name} must be contiguous")
    if f32 and t.dtype != _torch().float32:
        raise TypeError(f"{name} must be float32")
    if like is not None and (t.shape != like.shape or t.dtype != like.dtype or t.device != like.device):
        raise ValueError(f"{name} must match q in shape, dtype and device")
    return t.data_ptr()


_torch_mod = None


def _torch():
    global _torch_mod
    if _torch_mod is None:
        import torch
        _torch_mod = torch
    return _torch_mod


def _stream_handle(stream, device) -> int:
    if stream is None:
        return _torch().cuda.current_stream(device).cuda_stream
    return stream.cuda_stream if hasattr(stream, "cuda_stream") else int(stream)


class _alloc_on:
    """Allocate from torch's caching allocator as work of `stream`: a block handed out under
    another stream could be given to other work while the kernels enqueued on `stream` still use
    it.  `stream` = None (the current stream) needs nothing."""

    def __init__(self, stream, device):
        torch = _torch()
        if stream is None:
            self.ctx = None
        else:
            ts = stream if hasattr(stream, "cuda_stream") else torch.cuda.ExternalStream(int(stream), device=device)
            self.ctx = torch.cuda.stream(ts)

    def __enter__(self):
        if self.ctx is not None:
            self.ctx.__enter__()

    def __exit__(self, *exc):
        if self.ctx is not None:
            self.ctx.__exit__(*exc)


class _on_device:
    """Make `device` current for the duration of the call, only if it is not already."""

    def __init__(self, device):
        torch = _torch()
        self.ctx = None if device.index == torch.cuda.current_device() else torch.cuda.device(device)

    def __enter__(self):
        if self.ctx is not None:
            self.ctx.__enter__()

    def __exit__(self, *exc):
        if self.ctx is not None:
            self.ctx.__exit__(*exc)


def _bias_ptr(bias, heads: int, L: int):
    """(device pointer, dtype code) of a [heads, L, L] bias, fp32 or bf16."""
    if bias is None:
        return None, FWA_F32
    if tuple(bias.shape) != (heads, L, L):
        raise ValueError("bias must be [heads, L, L]")
    if bias.dtype == _torch().bfloat16:
        return _dev_ptr(bias, "bias"), FWA_BF16
    return _dev_ptr(bias, "bias", f32=True), FWA_F32


_native_mod = None


def _native():
    """The native marshalling module, linked against the ``libfwa.so`` beside it."""
    global _native_mod
    if _native_mod is None:
        load_library()
        _torch()
        try:
            from . import _fwa_torch
        except ImportError as e:
            raise RuntimeError(f"{os.path.join(_HERE, '_fwa_torch.so')} cannot be loaded ({e}): build it with "
                               "`python -m paper_2501_06480_amd.build`. There is no fallback path.") from e
        _native_mod = _fwa_torch
    return _native_mod


def _entry(what: str, bias, labels) -> str:
    """Name of the C entry a call went through, for the message of an error."""
    return what + ("_labels" if labels is not None or (bias is not None and bias.dtype == _torch().bfloat16) else "_strided")


def fwa_forward(q, k, v, heads: int, scale: float, bias=None, mask=None, out=None, stream=None, labels=None,
                mask_value: float = -100.0):
    """O = softmax(scale*QK^T + B + M) V (paper Algorithm 1).  Tensors are [N, L, C] on the GPU;
    q, k, v (and `out`) may be row-strided views, e.g. of a fused [N, L, 3, heads, d] tensor.
    The mask is a dense [nW, L, L] fp32 tensor, or int32 region `labels` [nW, L] from which the
    kernels form M[i][j] = 0 if labels agree else `mask_value`."""
    call = (_native_mod or _native()).forward
    if stream is None:
        o = call(q, k, v, int(heads), float(scale), bias, mask, out, None, labels, float(mask_value))
    else:
        with _alloc_on(stream, q.device):
            o = call(q, k, v, int(heads), float(scale), bias, mask, out, _stream_handle(stream, q.device), labels,
                     float(mask_value))
    if type(o) is int:
        raise FwaError(o, _entry("fwa_forward", bias, labels))
    return o


def fwa_forward_qkv(qkv, scale: float, bias=None, mask=None, labels=None, mask_value: float = -100.0):
    """``fwa_forward`` of the three slices of a contiguous fused [N, L, 3, heads, d] tensor, read in place."""
    o = (_native_mod or _native()).forward_qkv(qkv, float(scale), bias, mask, labels, float(mask_value))
    if type(o) is int:
        raise FwaError(o, _entry("fwa_forward", bias, labels))
    return o


def fwa_backward_workspace_bytes(N: int, L: int, C: int, heads: int, dtype: int, want_dbias: bool) -> int:
    return int(load_library().fwa_backward_workspace_bytes(N, L, C, heads, dtype, int(bool(want_dbias))))


def fwa_backward(q, k, v, d_o, heads: int, scale: float, bias=None, mask=None, want_dbias: bool = False,
                 workspace=None, stream=None, out=None, labels=None, mask_value: float = -100.0):
    """(dQ, dK, dV, dBias) from Q, K, V, dO (paper Algorithm 2).  dBias is None unless asked for.
    q, k, v, d_o may be row-strided views; `out` = (dq, dk, dv) writes the gradients into given
    tensors, e.g. the three views of a fused [N, L, 3, heads, d] gradient buffer.  `labels` and
    `mask_value` give the mask as region labels, as in ``fwa_forward``."""
    call = (_native_mod or _native()).backward
    dq, dk, dv = out if out is not None else (None, None, None)
    if stream is None:
        r = call(q, k, v, d_o, int(heads), float(scale), bias, mask, bool(want_dbias), workspace, None, dq, dk, dv, labels,
                 float(mask_value))
    else:
        with _alloc_on(stream, q.device):
            r = call(q, k, v, d_o, int(heads), float(scale), bias, mask, bool(want_dbias), workspace,
                     _stream_handle(stream, q.device), dq, dk, dv, labels, float(mask_value))
    if type(r) is int:
        raise FwaError(r, _entry("fwa_backward", bias, labels))
    return r


def fwa_backward_qkv(qkv, d_o, scale: float, bias=None, mask=None, want_dbias: bool = False, labels=None,
                     mask_value: float = -100.0):
    """(dqkv, dBias) of ``fwa_forward_qkv``: the gradients of the three slices written into one tensor like qkv."""
    r = (_native_mod or _native()).backward_qkv(qkv, d_o, float(scale), bias, mask, bool(want_dbias), labels, float(mask_value))
    if type(r) is int:
        raise FwaError(r, _entry("fwa_backward", bias, labels))
    return r


def fwa_backward_noalloc(q, k, v, d_o, heads: int, scale: float, out, dbias=None, bias=None, mask=None, stream=None):
    """``fwa_backward`` for callers that cannot allocate: the caller passes every output
    (`out` = (dq, dk, dv), contiguous; `dbias` = a [heads, L, L] fp32 tensor or None) and the
    library uses its own static scratch array as workspace.  Returns (dq, dk, dv, dbias)."""
    lib = load_library()
    N, L, C = q.shape
    dq, dk, dv = out
    nW = 0 if mask is None else int(mask.shape[0])
    if mask is not None and tuple(mask.shape) != (nW, L, L):
        raise ValueError("mask must be [nW, L, L]")
    if dbias is not None and tuple(dbias.shape) != (heads, L, L):
        raise ValueError("dbias must be [heads, L, L]")
    bp, bias_code = _bias_ptr(bias, heads, L)
    if bias_code != FWA_F32:
        raise TypeError("fwa_backward_noalloc takes an fp32 bias")
    args = (_dev_ptr(q, "q"), _dev_ptr(k, "k", q), _dev_ptr(v, "v", q), _dev_ptr(d_o, "d_o", q),
            _dev_ptr(dq, "dq", q), _dev_ptr(dk, "dk", q), _dev_ptr(dv, "dv", q), _dev_ptr(dbias, "dbias", f32=True),
            N, L, C, int(heads), float(scale), bp, _dev_ptr(mask, "mask", f32=True), nW, _dtype_code(q),
            _stream_handle(stream, q.device))
    with _on_device(q.device):
        rc = lib.fwa_backward_noalloc(*args)
    if rc != FWA_OK:
        raise FwaError(rc, "fwa_backward_noalloc")
    return dq, dk, dv, dbias


def _bias_call(fn, t, k: int, stream, what: str):
    call = getattr(_native_mod or _native(), fn)
    r = call(t, int(k), None if stream is None else _stream_handle(stream, t.device))
    if type(r) is int:
        raise FwaError(r, what)
    return r


def fwa_bias_gather(table, k: int, stream=None):
    """[heads, (2k-1)^2] fp32 table -> [heads, k*k, k*k] fp32 bias, on the GPU."""
    return _bias_call("bias_gather", table, k, stream, "fwa_bias_gather")


def fwa_bias_scatter(dbias, k: int, stream=None):
    """[heads, k*k, k*k] fp32 bias gradient -> [heads, (2k-1)^2] table gradient."""
    return _bias_call("bias_scatter", dbias, k, stream, "fwa_bias_scatter")
