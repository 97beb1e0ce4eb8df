"""Thin binding over libmonarch.so: argument marshalling only.

Every function has the name of the C entry point it calls (``include/monarch.h``).
PyTorch supplies device memory and the current HIP stream; all arithmetic runs in
the library's kernels.  The calls on tensors go through the native module ``_native``
(``csrc/monarch_torch.cpp``: checks, allocation, stream, call), which keeps their host
time at a few microseconds; the rest is ctypes.  There is no fallback: if either
library is missing, loading fails with an error that says how to build it.
"""
from __future__ import annotations

import ctypes
import os

import torch

_HERE = os.path.dirname(os.path.abspath(__file__))
LIB_PATH = os.path.join(_HERE, "libmonarch.so")

MONARCH_F32 = 0
MONARCH_BF16 = 1
MONARCH_OK = 0
MONARCH_ERR_INVALID = -1
MONARCH_ERR_UNSUPPORTED = -2
MONARCH_ERR_WORKSPACE = -3
MONARCH_ERR_HIP = -4
MONARCH_FLAG_WGRAD_F32 = 1
MONARCH_FLAG_PERM_B = 2
MONARCH_FLAG_GENERIC = 4
MONARCH_FLAG_WS_PACKED = 8

# every symbol include/monarch.h declares
EXPORTS = (
    "monarch_fwd", "monarch_fwd_ex", "monarch_fwd_ws", "monarch_fwd_static", "monarch_fwd_bias", "monarch_fwd_workspace_bytes",
    "monarch_fwd_packed", "monarch_fwd_packed_scratch_bytes", "monarch_bwd",
    "monarch_bwd_bias", "monarch_fwd_bias_gelu", "monarch_bwd_bias_gelu_in",
    "monarch_bwd_workspace_bytes",
    "monarch_fwd_t", "monarch_fwd_t_workspace_bytes", "monarch_saved_bytes", "monarch_fwd_save", "monarch_fwd_bias_save", "monarch_bwd_saved", "monarch_kept_bytes", "monarch_fwd_keep", "monarch_bwd_kept", "monarch_bwd_kept_workspace_bytes", "monarch_fwd_c64", "monarch_fwd_h_c64", "monarch_bwd_c64", "monarch_fwd_c64_ws", "monarch_fwd_h_c64_ws", "monarch_bwd_c64_ws", "monarch_c64_workspace_bytes", "monarch_dft_factors", "monarch_to_dense", "monarch_project", "monarch_kernel_name", "monarch_status_string", "monarch_version", "monarch_stream_copy", "monarch_launch_probe",
)

_lib = None


class MonarchError(RuntimeError):
    def __init__(self, status: int, where: str):
        self.status = status
        super().__init__("%s failed: %d (%s)" % (where, status, monarch_status_string(status)))


def lib() -> ctypes.CDLL:
    """Load libmonarch.so (built in-tree by ``paper_2204_00595_amd.build``)."""
    global _lib
    if _lib is None:
        if not os.path.exists(LIB_PATH):
            raise ImportError(
                "%s is missing: build it with `python -m paper_2204_00595_amd.build` "
                "(or __graft_entry__.build()); there is no fallback path" % LIB_PATH)
        L = ctypes.CDLL(LIB_PATH)
        vp, i64, ci, cu, sz = ctypes.c_void_p, ctypes.c_int64, ctypes.c_int, ctypes.c_uint, ctypes.c_size_t
        L.monarch_fwd.restype = ci
        L.monarch_fwd.argtypes = [vp, vp, vp, vp, i64, ci, ci, ci, ci, ci, vp]
        L.monarch_fwd_ex.restype = ci
        L.monarch_fwd_ex.argtypes = [vp, vp, vp, vp, i64, ci, ci, ci, ci, ci, vp, cu]
        L.monarch_fwd_ws.restype = ci
        L.monarch_fwd_ws.argtypes = [vp, vp, vp, vp, i64, ci, ci, ci, ci, ci, vp, vp, sz, cu]
        L.monarch_fwd_static.restype = ci
        L.monarch_fwd_static.argtypes = [vp, vp, vp, vp, i64, ci, ci, ci, ci, ci, vp, cu]
        L.monarch_fwd_bias.restype = ci
        L.monarch_fwd_bias.argtypes = [vp, vp, vp, vp, vp, i64, ci, ci, ci, ci, ci, vp, vp, sz, cu]
        L.monarch_fwd_packed.restype = ci
        L.monarch_fwd_packed.argtypes = [vp] * 4 + [ci, vp, vp, i64, ci, ci, ci, ci, ci, vp, vp, sz, vp, sz, cu]
        L.monarch_fwd_packed_scratch_bytes.restype = sz
        L.monarch_fwd_packed_scratch_bytes.argtypes = [i64, ci, ci, ci, ci, ci, cu]
        L.monarch_bwd_bias.restype = ci
        L.monarch_bwd_bias.argtypes = [vp] * 8 + [i64, ci, ci, ci, ci, ci, vp, vp, sz, cu]
        L.monarch_fwd_bias_gelu.restype = ci
        L.monarch_fwd_bias_gelu.argtypes = [vp] * 6 + [i64, ci, ci, ci, ci, ci, vp, vp, sz, cu]
        L.monarch_bwd_bias_gelu_in.restype = ci
        L.monarch_bwd_bias_gelu_in.argtypes = [vp] * 9 + [i64, ci, ci, ci, ci, ci, vp, vp, sz, cu]
        L.monarch_fwd_workspace_bytes.restype = sz
        L.monarch_fwd_workspace_bytes.argtypes = [i64, ci, ci, ci, ci, ci, cu]
        L.monarch_bwd.restype = ci
        L.monarch_bwd.argtypes = [vp] * 7 + [i64, ci, ci, ci, ci, ci, vp, vp, sz, cu]
        L.monarch_bwd_workspace_bytes.restype = sz
        L.monarch_bwd_workspace_bytes.argtypes = [i64, ci, ci, ci, ci, ci, cu]
        L.monarch_to_dense.restype = ci
        L.monarch_to_dense.argtypes = [vp, vp, vp, ci, ci, ci, ci, ci, vp, cu]
        L.monarch_fwd_t.restype = ci
        L.monarch_fwd_t.argtypes = [vp, vp, vp, vp, i64, ci, ci, ci, ci, ci, vp, vp, sz, cu]
        L.monarch_fwd_t_workspace_bytes.restype = sz
        L.monarch_fwd_t_workspace_bytes.argtypes = [i64, ci, ci, ci, ci, ci, cu]
        L.monarch_saved_bytes.restype = sz
        L.monarch_saved_bytes.argtypes = [i64, ci, ci, ci, ci, ci, cu]
        L.monarch_fwd_save.restype = ci
        L.monarch_fwd_save.argtypes = [vp, vp, vp, vp, vp, sz, i64, ci, ci, ci, ci, ci, vp, cu]
        L.monarch_fwd_bias_save.restype = ci
        L.monarch_fwd_bias_save.argtypes = [vp, vp, vp, vp, vp, vp, sz, i64, ci, ci, ci, ci, ci, vp, cu]
        L.monarch_bwd_saved.restype = ci
        L.monarch_bwd_saved.argtypes = [vp, vp, vp, sz, vp, vp, vp, vp, vp, vp, i64, ci, ci, ci, ci, ci, vp, vp, sz, cu]
        L.monarch_kept_bytes.restype = sz
        L.monarch_kept_bytes.argtypes = L.monarch_saved_bytes.argtypes
        L.monarch_fwd_keep.restype = ci
        L.monarch_fwd_keep.argtypes = L.monarch_fwd_bias_save.argtypes
        L.monarch_bwd_kept.restype = ci
        L.monarch_bwd_kept.argtypes = L.monarch_bwd_saved.argtypes
        L.monarch_bwd_kept_workspace_bytes.restype = sz
        L.monarch_bwd_kept_workspace_bytes.argtypes = L.monarch_saved_bytes.argtypes
        L.monarch_fwd_c64.restype = ci
        L.monarch_fwd_c64.argtypes = [vp, vp, vp, vp, i64, ci, ci, ci, ci, vp, cu]
        L.monarch_fwd_h_c64.restype = ci
        L.monarch_fwd_h_c64.argtypes = [vp, vp, vp, vp, i64, ci, ci, ci, ci, vp, cu]
        L.monarch_bwd_c64.restype = ci
        L.monarch_bwd_c64.argtypes = [vp] * 7 + [i64, ci, ci, ci, ci, vp, cu]
        L.monarch_bwd_c64_ws.restype = ci
        L.monarch_bwd_c64_ws.argtypes = [vp] * 7 + [i64, ci, ci, ci, ci, vp, vp, sz, cu]
        L.monarch_fwd_c64_ws.restype = ci
        L.monarch_fwd_c64_ws.argtypes = [vp, vp, vp, vp, i64, ci, ci, ci, ci, vp, vp, sz, cu]
        L.monarch_fwd_h_c64_ws.restype = ci
        L.monarch_fwd_h_c64_ws.argtypes = [vp, vp, vp, vp, i64, ci, ci, ci, ci, vp, vp, sz, cu]
        L.monarch_c64_workspace_bytes.restype = sz
        L.monarch_c64_workspace_bytes.argtypes = [ci, i64, ci, ci, ci, ci, cu]
        L.monarch_dft_factors.restype = ci
        L.monarch_dft_factors.argtypes = [vp, vp, ci, ci, vp]
        L.monarch_project.restype = ci
        L.monarch_project.argtypes = [vp, vp, vp, ci, ci, ci, vp, cu]
        L.monarch_kernel_name.restype = ctypes.c_char_p
        L.monarch_kernel_name.argtypes = [ci, ci, ci, ci, ci, ci, cu]
        L.monarch_status_string.restype = ctypes.c_char_p
        L.monarch_status_string.argtypes = [ci]
        L.monarch_version.restype = ci
        L.monarch_version.argtypes = []
        L.monarch_stream_copy.restype = ci
        L.monarch_stream_copy.argtypes = [vp, vp, sz, vp]
        L.monarch_launch_probe.restype = ci
        L.monarch_launch_probe.argtypes = [vp]
        _lib = L
    return _lib


class _Native:
    """The native module, loaded at the first call (so that this module imports before anything is built)."""

    def __getattr__(self, name):
        lib()  # the ImportError that says how to build, if nothing is
        try:
            from . import _native as m
        except ImportError as e:
            raise ImportError("%s: build it with `python -m paper_2204_00595_amd.build` (or __graft_entry__.build()); "
                              "there is no fallback path" % e) from e
        m.set_error(MonarchError)
        for f in dir(m):
            if not f.startswith("_"):
                setattr(self, f, getattr(m, f))
        return getattr(m, name)


_native_calls = _Native()


def _stream_ptr(stream) -> int:
    st = torch.cuda.current_stream() if stream is None else stream
    return int(st.cuda_stream)


def monarch_stream_copy(dst: torch.Tensor, src: torch.Tensor, stream=None) -> torch.Tensor:
    """Plain streaming copy src -> dst (same byte size, contiguous, on one GPU): the measured HBM roof."""
    nbytes = src.numel() * src.element_size()
    if dst.numel() * dst.element_size() != nbytes or not (dst.is_cuda and src.is_cuda and dst.device == src.device):
        raise ValueError("dst and src must be GPU tensors of the same byte size on one device")
    if not (dst.is_contiguous() and src.is_contiguous()):
        raise ValueError("dst and src must be contiguous")
    with torch.cuda.device(src.device):
        rc = lib().monarch_stream_copy(dst.data_ptr(), src.data_ptr(), nbytes, _stream_ptr(stream))
    if rc != MONARCH_OK:
        raise MonarchError(rc, "monarch_stream_copy")
    return dst


def monarch_launch_probe(stream=None) -> None:
    """Enqueue one empty kernel on the stream (the launch floor of the machine, for the benchmark)."""
    rc = lib().monarch_launch_probe(_stream_ptr(stream))
    if rc != MONARCH_OK:
        raise MonarchError(rc, "monarch_launch_probe")


def monarch_version() -> int:
    return int(lib().monarch_version())


def monarch_status_string(status: int) -> str:
    return lib().monarch_status_string(int(status)).decode()


def monarch_kernel_name(pass_: int, n_in: int, k: int, q: int, s: int, dtype: int, flags: int = 0) -> str:
    return lib().monarch_kernel_name(pass_, n_in, k, q, s, dtype, flags).decode()


def monarch_bwd_workspace_bytes(batch: int, n_in: int, k: int, q: int, s: int, dtype: int, flags: int = 0) -> int:
    return int(lib().monarch_bwd_workspace_bytes(batch, n_in, k, q, s, dtype, flags))


def monarch_fwd_workspace_bytes(batch: int, n_in: int, k: int, q: int, s: int, dtype: int, flags: int = 0) -> int:
    return int(lib().monarch_fwd_workspace_bytes(batch, n_in, k, q, s, dtype, flags))


def monarch_fwd_ws(x: torch.Tensor, R: torch.Tensor, L: torch.Tensor, y: torch.Tensor | None = None,
                   workspace: torch.Tensor | None = None, flags: int = 0, stream=None) -> torch.Tensor:
    """y = x M^T through monarch_fwd_ws.  The workspace is allocated when not given.

    With MONARCH_FLAG_WS_PACKED a workspace of packed weights is only read, here and in monarch_fwd_bias and
    monarch_fwd_bias_gelu: calls on several streams may share it.  What short batches need beside it is taken from the
    caching allocator for the call's stream (monarch_fwd_packed)."""
    return _native_calls.fwd_ws(x, R, L, y, workspace, flags, stream)


MONARCH_STATIC_WORKSPACE_BYTES = 8 << 20


def monarch_fwd_static(x: torch.Tensor, R: torch.Tensor, L: torch.Tensor, y: torch.Tensor, flags: int = 0,
                       stream=None) -> torch.Tensor:
    """y = x M^T through monarch_fwd_static (the library's own static workspace; nothing is allocated,
    so `y` must be given)."""
    return _native_calls.fwd_static(x, R, L, y, flags, stream)


def monarch_fwd(x: torch.Tensor, R: torch.Tensor, L: torch.Tensor, y: torch.Tensor | None = None,
                flags: int = 0, stream=None) -> torch.Tensor:
    """y = x M^T.  x (B, k*p), R (k, q, p), L (k, s, q) on the GPU; returns y (B, k*s)."""
    return _native_calls.fwd(x, R, L, y, flags, stream)


def monarch_to_dense(R: torch.Tensor, L: torch.Tensor, M: torch.Tensor | None = None, flags: int = 0,
                     stream=None) -> torch.Tensor:
    """M = P L P^T R as a dense (k*s, k*p) matrix.  R (k, q, p), L (k, s, q) on the GPU."""
    return _native_calls.to_dense(R, L, M, flags, stream)


def monarch_bwd(dy: torch.Tensor, x: torch.Tensor, R: torch.Tensor, L: torch.Tensor,
                dx: torch.Tensor | None = None, dR: torch.Tensor | None = None, dL: torch.Tensor | None = None,
                workspace: torch.Tensor | None = None, flags: int = 0, stream=None):
    """(dx, dR, dL) for upstream gradient dy (B, k*s).  Buffers are allocated when not given."""
    return _native_calls.bwd("monarch_bwd", dy, x, None, None, R, L, dx, dR, dL, None, False, workspace, flags, stream)[:3]


def monarch_fwd_bias(x: torch.Tensor, R: torch.Tensor, L: torch.Tensor, bias: torch.Tensor,
                     y: torch.Tensor | None = None, workspace: torch.Tensor | None = None, flags: int = 0,
                     stream=None) -> torch.Tensor:
    """y = x M^T + bias.  bias (k*s,) of the same dtype; the workspace is allocated when not given."""
    return _native_calls.fwd_bias(x, R, L, bias, y, workspace, flags, stream)


def monarch_bwd_bias(dy: torch.Tensor, x: torch.Tensor, R: torch.Tensor, L: torch.Tensor,
                     dx: torch.Tensor | None = None, dR: torch.Tensor | None = None, dL: torch.Tensor | None = None,
                     dbias: torch.Tensor | None = None, workspace: torch.Tensor | None = None, flags: int = 0,
                     stream=None):
    """(dx, dR, dL, dbias) for upstream gradient dy (B, k*s).  Buffers are allocated when not given."""
    return _native_calls.bwd("monarch_bwd_bias", dy, x, None, None, R, L, dx, dR, dL, dbias, True, workspace, flags, stream)


def monarch_fwd_bias_gelu(x: torch.Tensor, R: torch.Tensor, L: torch.Tensor, bias: torch.Tensor | None = None,
                          y_pre: torch.Tensor | None = None, y: torch.Tensor | None = None, want_pre: bool = True,
                          workspace: torch.Tensor | None = None, flags: int = 0, stream=None):
    """(y_pre, y) with y_pre = x M^T + bias and y = gelu(y_pre) (tanh form).  `want_pre=False` and no y_pre
    buffer: the pre-activation is not written and None is returned in its place."""
    return _native_calls.fwd_bias_gelu(x, R, L, bias, y_pre, y, want_pre, workspace, flags, stream)


def monarch_bwd_bias_gelu_in(dy: torch.Tensor, x: torch.Tensor, x_pre: torch.Tensor, R: torch.Tensor, L: torch.Tensor,
                             dx_pre: torch.Tensor | None = None, dR: torch.Tensor | None = None,
                             dL: torch.Tensor | None = None, dbias: torch.Tensor | None = None, want_dbias: bool = True,
                             workspace: torch.Tensor | None = None, flags: int = 0, stream=None):
    """(dx_pre, dR, dL, dbias) of the layer y = x M^T + bias whose input is x = gelu(x_pre): dx_pre is the
    gradient with respect to x_pre.  Buffers are allocated when not given."""
    if x_pre is None:
        raise TypeError("x_pre must be a tensor")
    return _native_calls.bwd("monarch_bwd_bias_gelu_in", dy, x, x_pre, None, R, L, dx_pre, dR, dL, dbias, want_dbias, workspace,
                             flags, stream)


def monarch_project(A: torch.Tensor, R: torch.Tensor | None = None, L: torch.Tensor | None = None, stream=None):
    """(L, R): factors of the square Monarch matrix closest to the dense A (n, n), n = m*m, m <= 64."""
    return _native_calls.project(A, R, L, stream)


def monarch_fwd_t_workspace_bytes(batch: int, n_in: int, k: int, q: int, s: int, dtype: int, flags: int = 0) -> int:
    return int(lib().monarch_fwd_t_workspace_bytes(batch, n_in, k, q, s, dtype, flags))


def monarch_fwd_t(x: torch.Tensor, R: torch.Tensor, L: torch.Tensor, y: torch.Tensor | None = None,
                  workspace: torch.Tensor | None = None, flags: int = 0, stream=None) -> torch.Tensor:
    """y = x M (the transposed Monarch matrix applied to the rows).  x (B, k*s) -> y (B, k*p)."""
    return _native_calls.fwd_t(x, R, L, y, workspace, flags, stream)


def monarch_saved_bytes(batch: int, n_in: int, k: int, q: int, s: int, dtype: int, flags: int = 0) -> int:
    return int(lib().monarch_saved_bytes(batch, n_in, k, q, s, dtype, flags))


def monarch_fwd_save(x: torch.Tensor, R: torch.Tensor, L: torch.Tensor, y: torch.Tensor | None = None,
                     saved: torch.Tensor | None = None, flags: int = 0, stream=None):
    """(y, saved): y = x M^T, and the buffer monarch_bwd_saved reads instead of recomputing (None when
    the shape has no such path)."""
    return _native_calls.fwd_save(x, R, L, None, y, saved, flags, stream)


def monarch_fwd_bias_save(x: torch.Tensor, R: torch.Tensor, L: torch.Tensor, bias: torch.Tensor, y: torch.Tensor | None = None,
                          saved: torch.Tensor | None = None, flags: int = 0, stream=None):
    """(y, saved) of the affine layer, y = x M^T + bias (saved is None when the shape has no such path)."""
    if bias is None:
        raise TypeError("bias must be a tensor")
    return _native_calls.fwd_save(x, R, L, bias, y, saved, flags, stream)


def monarch_bwd_saved(dy: torch.Tensor, x: torch.Tensor, saved: torch.Tensor | None, R: torch.Tensor, L: torch.Tensor,
                      dx: torch.Tensor | None = None, dR: torch.Tensor | None = None, dL: torch.Tensor | None = None,
                      dbias: torch.Tensor | None = None, want_dbias: bool = False,
                      workspace: torch.Tensor | None = None, flags: int = 0, stream=None):
    """(dx, dR, dL, dbias or None) with the vector saved by monarch_fwd_save (None: recompute)."""
    return _native_calls.bwd("monarch_bwd_saved", dy, x, None, saved, R, L, dx, dR, dL, dbias, want_dbias, workspace, flags, stream)


C64_FWD, C64_BWD, C64_FWD_H = 0, 1, 2


def monarch_c64_workspace_bytes(pass_: int, batch: int, n_in: int, k: int, q: int, s: int, flags: int = 0) -> int:
    """Workspace of monarch_fwd_c64_ws (C64_FWD), monarch_bwd_c64_ws (C64_BWD), monarch_fwd_h_c64_ws (C64_FWD_H)."""
    return int(lib().monarch_c64_workspace_bytes(pass_, batch, n_in, k, q, s, flags))


def monarch_fwd_c64(x: torch.Tensor, R: torch.Tensor, L: torch.Tensor, y: torch.Tensor | None = None,
                    flags: int = 0, stream=None) -> torch.Tensor:
    """y = x M^T for complex64 tensors (same shapes as monarch_fwd)."""
    return _native_calls.c64_apply(C64_FWD, False, x, R, L, y, None, flags, stream)


def monarch_fwd_h_c64(x: torch.Tensor, R: torch.Tensor, L: torch.Tensor, y: torch.Tensor | None = None,
                      flags: int = 0, stream=None) -> torch.Tensor:
    """y = x conj(M) (the conjugate transpose applied to every row) for complex64 tensors: x (B, k*s) -> y (B, k*p)."""
    return _native_calls.c64_apply(C64_FWD_H, False, x, R, L, y, None, flags, stream)


def monarch_bwd_c64(dy: torch.Tensor, x: torch.Tensor, R: torch.Tensor, L: torch.Tensor, flags: int = 0, stream=None):
    """(dx, dR, dL) for complex64 tensors, gradients in the dRe + i dIm convention."""
    return _native_calls.c64_bwd(False, dy, x, R, L, None, None, None, None, flags, stream)


def monarch_fwd_c64_ws(x: torch.Tensor, R: torch.Tensor, L: torch.Tensor, y: torch.Tensor | None = None,
                       workspace: torch.Tensor | None = None, flags: int = 0, stream=None) -> torch.Tensor:
    """monarch_fwd_c64 with a workspace (allocated when not given): matrix-core kernels for square blocks."""
    return _native_calls.c64_apply(C64_FWD, True, x, R, L, y, workspace, flags, stream)


def monarch_fwd_h_c64_ws(x: torch.Tensor, R: torch.Tensor, L: torch.Tensor, y: torch.Tensor | None = None,
                         workspace: torch.Tensor | None = None, flags: int = 0, stream=None) -> torch.Tensor:
    """monarch_fwd_h_c64 with a workspace (allocated when not given): matrix-core kernels for square blocks."""
    return _native_calls.c64_apply(C64_FWD_H, True, x, R, L, y, workspace, flags, stream)


def monarch_bwd_c64_ws(dy: torch.Tensor, x: torch.Tensor, R: torch.Tensor, L: torch.Tensor,
                       dx: torch.Tensor | None = None, dR: torch.Tensor | None = None, dL: torch.Tensor | None = None,
                       workspace: torch.Tensor | None = None, flags: int = 0, stream=None):
    """monarch_bwd_c64 with a workspace (allocated when not given): matrix-core kernels for square blocks, else
    the weight gradients contracted by a GEMM over operands kept in the workspace."""
    return _native_calls.c64_bwd(True, dy, x, R, L, dx, dR, dL, workspace, flags, stream)


def monarch_dft_factors(m: int, inverse: bool = False, device="cuda", stream=None):
    """(R, L): complex64 factors with P L P^T R = F_n P (n = m*m), or its inverse."""
    dev = torch.device(device)
    R = torch.empty((m, m, m), dtype=torch.complex64, device=dev)
    L = torch.empty((m, m, m), dtype=torch.complex64, device=dev)
    with torch.cuda.device(dev):
        rc = lib().monarch_dft_factors(R.data_ptr(), L.data_ptr(), m, 1 if inverse else 0, _stream_ptr(stream))
    if rc != MONARCH_OK:
        raise MonarchError(rc, "monarch_dft_factors")
    return R, L
