"""ctypes binding of the C-ABI attention library (include/qm_attn.h).

Argument marshalling only: every step of the attention forward runs in the
gfx950 kernels.  PyTorch supplies device memory and the current HIP stream.
There is no fallback: if ``libqm_attn.so`` is missing, loading fails loudly.
"""
from __future__ import annotations

import ctypes
import os
import threading

PKG_DIR = os.path.dirname(os.path.abspath(__file__))
LIB_PATH = os.path.join(PKG_DIR, "libqm_attn.so")
DEBUG_LIB_PATH = os.path.join(PKG_DIR, "libqm_attn_debug.so")

# qm_dtype_t
QM_F16 = 0
QM_BF16 = 1

# qm_layout_t
QM_BHND = 0
QM_BNHD = 1

# status codes
QM_OK = 0
QM_ERR_NULL = -1
QM_ERR_SHAPE = -2
QM_ERR_HEADDIM = -3
QM_ERR_DTYPE = -4
QM_ERR_SCALE = -5
QM_ERR_ALIAS = -6
QM_ERR_CAUSAL = -7
QM_ERR_LAUNCH = -8
QM_ERR_UNSUPPORTED = -9
QM_ERR_LAYOUT = -10
QM_ERR_TILE = -11

_lib = None
_lock = threading.Lock()


class QmAttnError(RuntimeError):
    """A non-zero status from the C library."""

    def __init__(self, status: int, message: str):
        super().__init__(f"qm_attn_fwd failed with status {status}: {message}")
        self.status = status


def _declare(lib: ctypes.CDLL) -> ctypes.CDLL:
    """Argument and result types of every entry point of ``include/qm_attn.h``."""
    lib.qm_attn_fwd.argtypes = [
        ctypes.c_void_p, ctypes.c_void_p, ctypes.c_void_p, ctypes.c_void_p, ctypes.c_void_p,
        ctypes.c_int, ctypes.c_int, ctypes.c_int, ctypes.c_int,
        ctypes.c_float, ctypes.c_int, ctypes.c_void_p, ctypes.c_int,
    ]
    lib.qm_attn_fwd.restype = ctypes.c_int
    lib.qm_attn_fwd_gqa.argtypes = [
        ctypes.c_void_p, ctypes.c_void_p, ctypes.c_void_p, ctypes.c_void_p, ctypes.c_void_p,
        ctypes.c_int, ctypes.c_int, ctypes.c_int, ctypes.c_int, ctypes.c_int,
        ctypes.c_float, ctypes.c_int, ctypes.c_void_p, ctypes.c_int,
    ]
    lib.qm_attn_fwd_gqa.restype = ctypes.c_int
    lib.qm_attn_fwd_mla.argtypes = [
        ctypes.c_void_p, ctypes.c_void_p, ctypes.c_void_p, ctypes.c_void_p, ctypes.c_void_p,
        ctypes.c_int, ctypes.c_int, ctypes.c_int, ctypes.c_int, ctypes.c_int,
        ctypes.c_float, ctypes.c_int, ctypes.c_void_p, ctypes.c_int,
    ]
    lib.qm_attn_fwd_mla.restype = ctypes.c_int
    lib.qm_attn_fwd_fp8.argtypes = [
        ctypes.c_void_p, ctypes.c_void_p, ctypes.c_void_p, ctypes.c_void_p, ctypes.c_void_p,
        ctypes.c_int, ctypes.c_int, ctypes.c_int, ctypes.c_int,
        ctypes.c_float, ctypes.c_float, ctypes.c_float, ctypes.c_float, ctypes.c_int,
        ctypes.c_void_p,
    ]
    lib.qm_attn_fwd_fp8.restype = ctypes.c_int
    lib.qm_attn_fwd_layout.argtypes = [
        ctypes.c_void_p, ctypes.c_void_p, ctypes.c_void_p, ctypes.c_void_p, ctypes.c_void_p,
        ctypes.c_int, ctypes.c_int, ctypes.c_int, ctypes.c_int, ctypes.c_int, ctypes.c_int,
        ctypes.c_float, ctypes.c_int, ctypes.c_void_p, ctypes.c_int, ctypes.c_int,
    ]
    lib.qm_attn_fwd_layout.restype = ctypes.c_int
    lib.qm_attn_fwd_fp8_layout.argtypes = [
        ctypes.c_void_p, ctypes.c_void_p, ctypes.c_void_p, ctypes.c_void_p, ctypes.c_void_p,
        ctypes.c_int, ctypes.c_int, ctypes.c_int, ctypes.c_int, ctypes.c_int,
        ctypes.c_float, ctypes.c_float, ctypes.c_float, ctypes.c_float, ctypes.c_int,
        ctypes.c_void_p, ctypes.c_int,
    ]
    lib.qm_attn_fwd_fp8_layout.restype = ctypes.c_int
    lib.qm_attn_set_tile_rows.argtypes = [ctypes.c_int]
    lib.qm_attn_set_tile_rows.restype = ctypes.c_int
    lib.qm_attn_strerror.argtypes = [ctypes.c_int]
    lib.qm_attn_strerror.restype = ctypes.c_char_p
    return lib


def load_library(path: str = LIB_PATH) -> ctypes.CDLL:
    """Load (once) and return the HIP library; raise if it has not been built."""
    global _lib
    if _lib is not None:
        return _lib
    with _lock:
        if _lib is not None:
            return _lib
        _lib = open_library(path)
        return _lib


def open_library(path: str) -> ctypes.CDLL:
    """A separate handle on a build of the library at ``path`` (the tests use
    it for the checking build, ``libqm_attn_debug.so``); raises if missing."""
    if not os.path.exists(path):
        raise RuntimeError(
            f"{path} is missing: the HIP attention library has not been built "
            "(run `python -m paper_2506_12355_amd.build`)")
    return _declare(ctypes.CDLL(path))


def strerror(status: int) -> str:
    return load_library().qm_attn_strerror(int(status)).decode()


def set_tile_rows(rows: int) -> None:
    """Query rows per workgroup for later calls: 0 (chosen from the shape, the
    default), 128 or 256.  Outputs are byte-identical either way; only speed
    changes (``qm_attn_set_tile_rows``)."""
    status = load_library().qm_attn_set_tile_rows(int(rows))
    if status != QM_OK:
        raise QmAttnError(status, strerror(status))


def qm_attn_fwd(q, k, v, o, lse, B, H, N, d, scale, causal, stream, dtype) -> int:
    """The C entry point with plain integers for pointers; returns the status."""
    return load_library().qm_attn_fwd(q, k, v, o, lse, int(B), int(H), int(N), int(d),
                                      float(scale), int(causal), stream, int(dtype))


def qm_attn_fwd_layout(q, k, v, o, lse, B, H, Hkv, N, d_qk, d_v, scale, causal, stream, dtype,
                       layout) -> int:
    """The general 16-bit C entry point (layout argument) with plain integers
    for pointers; returns the status."""
    return load_library().qm_attn_fwd_layout(q, k, v, o, lse, int(B), int(H), int(Hkv), int(N),
                                             int(d_qk), int(d_v), float(scale), int(causal),
                                             stream, int(dtype), int(layout))


def qm_attn_fwd_gqa(q, k, v, o, lse, B, H, Hkv, N, d, scale, causal, stream, dtype) -> int:
    """The grouped-query C entry point with plain integers for pointers; returns the status."""
    return load_library().qm_attn_fwd_gqa(q, k, v, o, lse, int(B), int(H), int(Hkv), int(N),
                                          int(d), float(scale), int(causal), stream, int(dtype))


def qm_attn_fwd_mla(q, k, v, o, lse, B, H, N, d_qk, d_v, scale, causal, stream, dtype) -> int:
    """The unequal-head-dimension C entry point with plain integers for pointers."""
    return load_library().qm_attn_fwd_mla(q, k, v, o, lse, int(B), int(H), int(N), int(d_qk),
                                          int(d_v), float(scale), int(causal), stream, int(dtype))


def qm_attn_fwd_fp8(q, k, v, o, lse, B, H, N, d, q_scale, k_scale, v_scale, scale, causal,
                    stream) -> int:
    """The FP8 C entry point with plain integers for pointers; returns the status."""
    return load_library().qm_attn_fwd_fp8(q, k, v, o, lse, int(B), int(H), int(N), int(d),
                                          float(q_scale), float(k_scale), float(v_scale),
                                          float(scale), int(causal), stream)


def fwd_fp8(q, k, v, scales, causal: bool = False, scale: float | None = None, out=None,
            lse=None, stream=None, layout: str = "bhnd"):
    """FP8 attention forward: q is [B, H, N, d], k and v [B, Hkv, N, d] (Hkv
    dividing H: grouped-query attention when Hkv < H) tensors of OCP E4M3 codes
    (``torch.float8_e4m3fn`` or ``uint8``) on a ROCm device; ``scales`` holds
    the three per-tensor factors (q_scale, k_scale, v_scale).  With
    ``layout="bnhd"`` the tensors are [B, N, heads, d] instead.  Returns
    (o, lse): o bf16 shaped like q, lse float32 [B, H, N] in either layout.
    ``scale`` defaults to 1/sqrt(d) rounded to float32.  Multi-head
    [B, H, N, d] calls go to ``qm_attn_fwd_fp8``, the others to
    ``qm_attn_fwd_fp8_layout``."""
    import torch

    if layout not in ("bhnd", "bnhd"):
        raise ValueError(f"layout must be 'bhnd' or 'bnhd', not {layout!r}")
    bnhd = layout == "bnhd"
    device = q.device
    for t in (q, k, v):
        if t.dim() != 4:
            names = "[B, N, H, d]" if bnhd else "[B, H, N, d]"
            raise ValueError(f"q, k and v must have shape {names}")
        if t.dtype not in (torch.uint8, torch.float8_e4m3fn):
            raise TypeError("FP8 inputs must be float8_e4m3fn or uint8 codes")
        if not t.is_cuda or t.device != device or not t.is_contiguous():
            raise ValueError("q, k and v must be contiguous tensors on one ROCm device")
    if bnhd:
        B, N, H, d = q.shape
        Bk, Nk, Hkv, dk = k.shape
    else:
        B, H, N, d = q.shape
        Bk, Hkv, Nk, dk = k.shape
    if v.shape != k.shape or Bk != B or Nk != N or dk != d:
        raise ValueError("k and v must hold Hkv heads matching q in B, N and d")
    scale = 1.0 / d ** 0.5 if scale is None else float(scale)   # rounded to float32 by the call
    if out is None:
        out = torch.empty(q.shape, dtype=torch.bfloat16, device=device)
    elif out.shape != q.shape or out.dtype != torch.bfloat16 or not out.is_contiguous():
        raise ValueError("out must be a contiguous bfloat16 tensor shaped like q")
    lse = _lse(q, lse, B, H, N)
    _check_outputs_on(device, out, lse)
    qs, ks, vs = (float(t) for t in scales)
    args = (q.data_ptr(), k.data_ptr(), v.data_ptr(), out.data_ptr(), lse.data_ptr(), B, H)
    if bnhd or Hkv != H:
        _enqueue(load_library().qm_attn_fwd_fp8_layout, device, stream,
                 args + (Hkv, N, d, qs, ks, vs, scale, 1 if causal else 0),
                 (QM_BNHD if bnhd else QM_BHND,))
    else:
        _enqueue(load_library().qm_attn_fwd_fp8, device, stream,
                 args + (N, d, qs, ks, vs, scale, 1 if causal else 0), ())
    return out, lse


def qm_attn_fwd_fp8_layout(q, k, v, o, lse, B, H, Hkv, N, d, q_scale, k_scale, v_scale, scale,
                           causal, stream, layout) -> int:
    """The general FP8 C entry point (key/value heads and layout as arguments)
    with plain integers for pointers; returns the status."""
    return load_library().qm_attn_fwd_fp8_layout(
        q, k, v, o, lse, int(B), int(H), int(Hkv), int(N), int(d), float(q_scale),
        float(k_scale), float(v_scale), float(scale), int(causal), stream, int(layout))


def _check_outputs_on(device, out, lse) -> None:
    """The kernel writes o and lse through device pointers: both must live on
    the inputs' device (a host tensor's address would be written by the GPU)."""
    for name, t in (("out", out), ("lse", lse)):
        if not t.is_cuda or t.device != device:
            raise ValueError(f"{name} must be on the inputs' device {device}, not {t.device}")


def _lse(q, lse, B, H, N):
    """The log-sum-exp output: the caller's, checked, or a new tensor."""
    import torch
    if lse is None:
        return torch.empty((B, H, N), dtype=torch.float32, device=q.device)
    if lse.shape != (B, H, N) or lse.dtype != torch.float32 or not lse.is_contiguous():
        raise ValueError("lse must be a contiguous float32 tensor of shape [B, H, N]")
    return lse


def _enqueue(entry, device, stream, before, after) -> None:
    """Call a C entry point (arguments before and after its stream) with `device`
    current, on `stream` (a torch stream; None: the device's current one)."""
    import torch
    index = device.index
    # the current stream's handle alone, without a torch.cuda.Stream object around it
    raw = torch._C._cuda_getCurrentRawStream(index) if stream is None else stream.cuda_stream
    if index == torch.cuda.current_device():
        status = entry(*before, raw, *after)
    else:
        with torch.cuda.device(index):
            status = entry(*before, raw, *after)
    if status != QM_OK:
        raise QmAttnError(status, strerror(status))


def _dtype_code(t) -> int:
    import torch
    if t.dtype == torch.float16:
        return QM_F16
    if t.dtype == torch.bfloat16:
        return QM_BF16
    raise TypeError(f"q, k, v must be float16 or bfloat16, not {t.dtype}")


def fwd(q, k, v, causal: bool = False, scale: float | None = None, out=None, lse=None,
        stream=None, layout: str = "bhnd"):
    """Attention forward on torch tensors on a ROCm device.

    q is [B, H, N, d]; k is [B, Hkv, N, d] and v [B, Hkv, N, dv] with Hkv
    dividing H.  Hkv = H and dv = d: multi-head attention (``qm_attn_fwd``);
    Hkv < H: grouped-query or multi-query attention (``qm_attn_fwd_gqa``);
    dv < d (d = 192, dv = 128, Hkv = H): the MLA shape (``qm_attn_fwd_mla``).
    With ``layout="bnhd"`` the tensors are [B, N, heads, width] instead (q
    [B, N, H, d], k [B, N, Hkv, d], v [B, N, Hkv, dv], o [B, N, H, dv];
    ``qm_attn_fwd_layout``).  Returns (o, lse): o of q's dtype, lse float32
    [B, H, N] in either layout.  ``scale`` defaults to 1/sqrt(d) rounded to
    float32.  ``stream`` defaults to the current stream of q's device.
    """
    import torch

    if layout not in ("bhnd", "bnhd"):
        raise ValueError(f"layout must be 'bhnd' or 'bnhd', not {layout!r}")
    bnhd = layout == "bnhd"
    if q.dim() != 4:
        raise ValueError(f"q must have shape {'[B, N, H, d]' if bnhd else '[B, H, N, d]'}")
    # a head's rows lie along `rows`, heads along `heads`
    rows, heads = (1, 2) if bnhd else (2, 1)
    qs, ks, vs = q.shape, k.shape, v.shape
    if len(ks) != 4 or len(vs) != 4 or vs[:3] != ks[:3]:
        raise ValueError("k must hold Hkv heads of width d and v Hkv heads of width dv")
    B, H, N, d = qs[0], qs[heads], qs[rows], qs[3]
    Hkv, dv = ks[heads], vs[3]
    if ks[0] != B or ks[rows] != N or ks[3] != d:
        raise ValueError("k must match q in B, N and d")
    if not (q.is_cuda and k.is_cuda and v.is_cuda):
        raise ValueError("q, k and v must be on a ROCm device")
    device = q.device
    if not (device == k.device == v.device):
        raise ValueError("q, k and v must be on the same device")
    if not (q.dtype == k.dtype == v.dtype):
        raise TypeError("q, k and v must have the same dtype")
    if not (q.is_contiguous() and k.is_contiguous() and v.is_contiguous()):
        names = "[B, N, H, d]" if bnhd else "[B, H, N, d]"
        raise ValueError(f"q, k and v must be contiguous {names}")
    code = _dtype_code(q)
    # the C float argument rounds the scale to float32
    scale = 1.0 / d ** 0.5 if scale is None else float(scale)
    if out is None:
        out = torch.empty((*qs[:3], dv), dtype=q.dtype, device=device)
    else:
        oshape = (*qs[:3], dv)
        if tuple(out.shape) != oshape or out.dtype != q.dtype or not out.is_contiguous():
            raise ValueError(f"out must be a contiguous {list(oshape)} tensor of q's dtype")
    lse = _lse(q, lse, B, H, N)
    _check_outputs_on(device, out, lse)
    lib = load_library()
    args = (q.data_ptr(), k.data_ptr(), v.data_ptr(), out.data_ptr(), lse.data_ptr(), B, H)
    causal = 1 if causal else 0
    if bnhd:
        _enqueue(lib.qm_attn_fwd_layout, device, stream, args + (Hkv, N, d, dv, scale, causal),
                 (code, QM_BNHD))
    elif dv != d:
        if Hkv != H:
            raise ValueError("unequal head dimensions need as many key/value heads as query heads")
        _enqueue(lib.qm_attn_fwd_mla, device, stream, args + (N, d, dv, scale, causal), (code,))
    elif Hkv == H:
        _enqueue(lib.qm_attn_fwd, device, stream, args + (N, d, scale, causal), (code,))
    else:
        _enqueue(lib.qm_attn_fwd_gqa, device, stream, args + (Hkv, N, d, scale, causal), (code,))
    return out, lse
