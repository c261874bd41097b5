"""Thin binding over libesc_convattn.so (include/esc_convattn.h).

Argument marshalling only: every step of the ConvAttn forward (Eq. 4 of the ESC
paper) runs in the HIP kernels.  torch supplies device memory and streams.  The calls
made once per pass check their tensors in native code (csrc/esc_native.cpp, built into
_native.so); the workspace calls, made once, go through ctypes.
There is no CPU fallback; a missing library raises.
"""
from __future__ import annotations

import ctypes
import importlib
import os
from typing import Optional

import torch

_HERE = os.path.dirname(os.path.abspath(__file__))
LIB_PATH = os.path.join(_HERE, "csrc", "libesc_convattn.so")
NATIVE_PATH = os.path.join(_HERE, "_native.so")

ESC_F32 = 0
ESC_BF16 = 1

EXPORTS = ("esc_workspace_bytes", "esc_workspace_init", "esc_workspace_errors", "esc_dynkernel_gen",
           "esc_convattn_forward", "esc_convattn_forward_noalloc", "esc_fused_workspace_bytes",
           "esc_convattn_fused_forward", "esc_dense_workspace_bytes", "esc_convattn_dense_forward",
           "esc_backward_workspace_bytes", "esc_convattn_backward", "esc_convffn_workspace_bytes",
           "esc_convffn_forward", "esc_residual_step_workspace_bytes", "esc_residual_step_forward", "esc_status_string")
NOALLOC_SCRATCH_BYTES = 1 << 20


class EscError(RuntimeError):
    def __init__(self, status: int, message: str):
        super().__init__(f"esc_convattn: status {status}: {message}")
        self.status = status


class _GenParams(ctypes.Structure):
    _fields_ = [("hidden", ctypes.c_int),
                ("w_down", ctypes.c_void_p), ("b_down", ctypes.c_void_p),
                ("w_up", ctypes.c_void_p), ("b_up", ctypes.c_void_p)]


class _GenGrads(ctypes.Structure):
    _fields_ = [("w_down", ctypes.c_void_p), ("b_down", ctypes.c_void_p),
                ("w_up", ctypes.c_void_p), ("b_up", ctypes.c_void_p)]


class _NativeModule:
    """Stands for the native half until a call needs it; raises (never falls back) when it is not built."""

    def __getattr__(self, name):
        global _native
        load_library()
        if not os.path.exists(NATIVE_PATH):
            raise FileNotFoundError(f"{NATIVE_PATH} is not built; run `python -m paper_2503_06671_amd.build` "
                                    "(or __graft_entry__.build()) first")
        _native = importlib.import_module("paper_2503_06671_amd._native")  # (one that is there and does not load says why)
        return getattr(_native, name)


_native = _NativeModule()
_lib = None


def load_library():
    """Load the built library; raise (never fall back) when it is missing."""
    global _lib
    if _lib is None:
        if not os.path.exists(LIB_PATH):
            raise FileNotFoundError(
                f"{LIB_PATH} is not built; run `python -m paper_2503_06671_amd.build` "
                "(or __graft_entry__.build()) first")
        lib = ctypes.CDLL(LIB_PATH)
        vp, ci, cl, sz = ctypes.c_void_p, ctypes.c_int, ctypes.c_long, ctypes.c_size_t
        lib.esc_workspace_bytes.argtypes = [ci, ci, ci, ci]
        lib.esc_workspace_bytes.restype = sz
        lib.esc_workspace_init.argtypes = [vp, sz, vp]
        lib.esc_workspace_init.restype = ci
        lib.esc_workspace_errors.argtypes = [vp, sz, vp, ctypes.POINTER(ctypes.c_uint)]
        lib.esc_workspace_errors.restype = ci
        lib.esc_dynkernel_gen.argtypes = [vp, ci, ci, ci, ci, ci, ci, ctypes.POINTER(_GenParams), vp,
                                          vp, sz, vp]
        lib.esc_dynkernel_gen.restype = ci
        lib.esc_convattn_forward.argtypes = [vp, ci, ci, ci, ci, ci, ci, vp, ci, cl,
                                             ctypes.POINTER(_GenParams), vp, vp, vp, sz, vp]
        lib.esc_convattn_forward.restype = ci
        lib.esc_convattn_forward_noalloc.argtypes = [vp, ci, ci, ci, ci, ci, ci, vp, ci, cl,
                                                     ctypes.POINTER(_GenParams), vp, vp, vp]
        lib.esc_convattn_forward_noalloc.restype = ci
        lib.esc_fused_workspace_bytes.argtypes = [ci, ci, ci, ci, ci, ci]
        lib.esc_fused_workspace_bytes.restype = sz
        lib.esc_convattn_fused_forward.argtypes = [vp, ci, ci, ci, ci, ci, ci, vp, vp, ci, cl,
                                                   ctypes.POINTER(_GenParams), vp, vp, vp, vp, vp, vp, sz, vp]
        lib.esc_convattn_fused_forward.restype = ci
        lib.esc_dense_workspace_bytes.argtypes = [ci, ci, ci, ci, ci]
        lib.esc_dense_workspace_bytes.restype = sz
        lib.esc_convattn_dense_forward.argtypes = [vp, ci, ci, ci, ci, ci, ci, vp, ci,
                                                   ctypes.POINTER(_GenParams), vp, vp, vp, sz, vp]
        lib.esc_convattn_dense_forward.restype = ci
        lib.esc_backward_workspace_bytes.argtypes = [ci, ci, ci, ci, ci, ci]
        lib.esc_backward_workspace_bytes.restype = sz
        lib.esc_convattn_backward.argtypes = [vp, vp, ci, ci, ci, ci, ci, ci, vp, ci, cl, ctypes.POINTER(_GenParams), vp,
                                              vp, vp, ctypes.POINTER(_GenGrads), vp, ci, vp, sz, vp]
        lib.esc_convattn_backward.restype = ci
        lib.esc_convffn_workspace_bytes.argtypes = [ci, ci, ci, ci, ci]
        lib.esc_convffn_workspace_bytes.restype = sz
        lib.esc_convffn_forward.argtypes = [vp, ci, ci, ci, ci, ci, ci, vp, vp, vp, vp, vp, vp, vp, vp, sz, vp]
        lib.esc_convffn_forward.restype = ci
        lib.esc_residual_step_workspace_bytes.argtypes = [ci, ci, ci, ci, ci, ci, ci, ci]
        lib.esc_residual_step_workspace_bytes.restype = sz
        lib.esc_residual_step_forward.argtypes = [vp, ci, ci, ci, ci, ci, ci, vp, vp, vp, vp, vp, vp, ci, vp, vp, ci, cl,
                                                  ctypes.POINTER(_GenParams), vp, vp, vp, vp, sz, vp]
        lib.esc_residual_step_forward.restype = ci
        lib.esc_status_string.argtypes = [ci]
        lib.esc_status_string.restype = ctypes.c_char_p
        _lib = lib
    return _lib


def status_string(status: int) -> str:
    return load_library().esc_status_string(int(status)).decode()


def _check(status: int) -> None:
    if status != 0:
        raise EscError(status, status_string(status))


def _ptr(t: Optional[torch.Tensor]) -> Optional[int]:
    return None if t is None else t.data_ptr()


def _stream(stream) -> Optional[int]:
    if stream is None:
        stream = torch.cuda.current_stream()
    return stream.cuda_stream or None


def _dev_f32(t: Optional[torch.Tensor], name: str) -> Optional[torch.Tensor]:
    if t is None:
        return None
    if not t.is_cuda or t.dtype != torch.float32 or not t.is_contiguous():
        raise TypeError(f"{name} must be a contiguous float32 device tensor")
    return t


class GenParams:
    """Device weights of the kernel estimator (Eq. 4 line 2); see esc_gen_params."""

    def __init__(self, w_up: torch.Tensor, b_up: Optional[torch.Tensor] = None, hidden: int = 0,
                 w_down: Optional[torch.Tensor] = None, b_down: Optional[torch.Tensor] = None):
        self.tensors = (_dev_f32(w_down, "w_down"), _dev_f32(b_down, "b_down"),
                        _dev_f32(w_up, "w_up"), _dev_f32(b_up, "b_up"))
        self.hidden = int(hidden)
        self.c = _GenParams(self.hidden, *[_ptr(t) for t in self.tensors])

    def __getattr__(self, name):
        # the native half's view of the weights, made at the first call that needs it (one, whichever thread is first)
        if name == "handle":
            return self.__dict__.setdefault(name, _native.gen_handle(self.hidden, *self.tensors))
        raise AttributeError(name)

    def check(self, Ca: int) -> None:
        """The library reads these buffers by the sizes C_a and hidden imply: refuse others."""
        w_down, b_down, w_up, b_up = self.tensors
        K = self.hidden if self.hidden > 0 else Ca
        want = {"w_up": (w_up, 9 * Ca * K), "b_up": (b_up, 9 * Ca)}
        if self.hidden > 0:
            want["w_down"] = (w_down, self.hidden * Ca)
            want["b_down"] = (b_down, self.hidden)
            if w_down is None:
                raise ValueError("hidden > 0 needs w_down")
        for name, (tensor, numel) in want.items():
            if tensor is not None and tensor.numel() != numel:
                raise ValueError(f"{name} has {tensor.numel()} elements, C_a = {Ca} and hidden = {self.hidden} "
                                 f"need {numel}")


def workspace_bytes(N: int, Ca: int, H: int, W: int) -> int:
    return int(load_library().esc_workspace_bytes(N, Ca, H, W))


def workspace_init(ws: torch.Tensor, stream=None) -> None:
    _check(load_library().esc_workspace_init(_ptr(ws), ws.numel() * ws.element_size(), _stream(stream)))


def workspace_errors(ws: torch.Tensor, stream=None) -> int:
    """Diagnostic: synchronises the stream and returns the workspace's error word."""
    v = ctypes.c_uint(0)
    _check(load_library().esc_workspace_errors(_ptr(ws), ws.numel() * ws.element_size(), _stream(stream),
                                               ctypes.byref(v)))
    return int(v.value)


def new_workspace(N: int, Ca: int, H: int, W: int, device="cuda", stream=None) -> torch.Tensor:
    """Allocate (with torch) and prepare a workspace for this shape."""
    nbytes = workspace_bytes(N, Ca, H, W)
    if nbytes == 0:
        raise ValueError("bad shape for a workspace")
    ws = torch.empty(nbytes, dtype=torch.uint8, device=device)
    workspace_init(ws, stream)
    return ws


def dynkernel_gen(x: torch.Tensor, Ca: int, gen: GenParams, workspace: torch.Tensor,
                  dk_out: Optional[torch.Tensor] = None, stream=None) -> torch.Tensor:
    """esc_dynkernel_gen: DK [N,Ca,3,3] float32 from GAP of the attention slice."""
    return _native.dynkernel_gen(x, Ca, gen, workspace, dk_out, stream)


def convattn_forward(x: torch.Tensor, Ca: int, lk: torch.Tensor, workspace: Optional[torch.Tensor],
                     gen: Optional[GenParams] = None, dk_in: Optional[torch.Tensor] = None,
                     out: Optional[torch.Tensor] = None, stream=None, ks: Optional[int] = None,
                     lk_channel_stride: Optional[int] = None) -> torch.Tensor:
    """esc_convattn_forward (workspace given) or esc_convattn_forward_noalloc (workspace None).
    lk is [Ca,Ks,Ks] (one filter per channel) or [Ks,Ks] (shared); with ks and
    lk_channel_stride given it is a flat buffer with channel c at c * stride."""
    return _native.convattn_forward(x, Ca, lk, workspace, gen, dk_in, out, stream, ks, lk_channel_stride)


def fused_workspace_bytes(N: int, Ca: int, H: int, W: int, dtype: torch.dtype, with_lk_c: bool) -> int:
    dt = ESC_F32 if dtype == torch.float32 else ESC_BF16
    return int(load_library().esc_fused_workspace_bytes(N, Ca, H, W, dt, int(bool(with_lk_c))))


def new_fused_workspace(N: int, Ca: int, H: int, W: int, dtype: torch.dtype, with_lk_c: bool, device="cuda",
                        stream=None) -> torch.Tensor:
    """Allocate (with torch) and prepare a workspace for esc_convattn_fused_forward."""
    nbytes = fused_workspace_bytes(N, Ca, H, W, dtype, with_lk_c)
    if nbytes == 0:
        raise ValueError("bad shape for a workspace")
    ws = torch.empty(nbytes, dtype=torch.uint8, device=device)
    workspace_init(ws, stream)
    return ws


def convattn_fused_forward(x: torch.Tensor, Ca: int, lk: torch.Tensor, w_fuse: torch.Tensor, workspace: torch.Tensor,
                           b_fuse: Optional[torch.Tensor] = None, lk_c: Optional[torch.Tensor] = None,
                           residual: Optional[torch.Tensor] = None, gen: Optional[GenParams] = None,
                           dk_in: Optional[torch.Tensor] = None, out: Optional[torch.Tensor] = None,
                           stream=None) -> torch.Tensor:
    """esc_convattn_fused_forward: the module with Conv_fuse, optionally LK^c and the residual."""
    return _native.convattn_fused_forward(x, Ca, lk, w_fuse, workspace, b_fuse, lk_c, residual, gen, dk_in, out, stream)


def new_convffn_workspace(N: int, Ch: int, H: int, W: int, dtype: torch.dtype, device="cuda") -> torch.Tensor:
    """Allocate (with torch) the scratch workspace of esc_convffn_forward (needs no preparation)."""
    dt = ESC_F32 if dtype == torch.float32 else ESC_BF16
    nbytes = int(load_library().esc_convffn_workspace_bytes(N, Ch, H, W, dt))
    if nbytes == 0:
        raise ValueError("bad shape for a workspace")
    return torch.empty(nbytes, dtype=torch.uint8, device=device)


def convffn_forward(x: torch.Tensor, w1: torch.Tensor, k_dw: torch.Tensor, w2: torch.Tensor, workspace: torch.Tensor,
                    b1: Optional[torch.Tensor] = None, b_dw: Optional[torch.Tensor] = None,
                    b2: Optional[torch.Tensor] = None, out: Optional[torch.Tensor] = None, stream=None) -> torch.Tensor:
    """esc_convffn_forward: w1 [Ch, C], k_dw [Ch, 3, 3], w2 [C, Ch], optional biases."""
    return _native.convffn_forward(x, w1, k_dw, w2, workspace, b1, b_dw, b2, out, stream)


def new_residual_step_workspace(N: int, C: int, H: int, W: int, Ca: int, Ch: int, dtype: torch.dtype, with_lk_c: bool,
                                device="cuda", stream=None) -> torch.Tensor:
    """Allocate (with torch) and prepare a workspace for esc_residual_step_forward."""
    dt = ESC_F32 if dtype == torch.float32 else ESC_BF16
    nbytes = int(load_library().esc_residual_step_workspace_bytes(N, C, H, W, Ca, Ch, dt, int(bool(with_lk_c))))
    if nbytes == 0:
        raise ValueError("bad shape for a workspace")
    ws = torch.empty(nbytes, dtype=torch.uint8, device=device)
    workspace_init(ws, stream)
    return ws


def residual_step_forward(f_in: torch.Tensor, w1: torch.Tensor, k_dw: torch.Tensor, w2: torch.Tensor, Ca: int,
                          lk: torch.Tensor, w_fuse: torch.Tensor, workspace: torch.Tensor,
                          b1: Optional[torch.Tensor] = None, b_dw: Optional[torch.Tensor] = None,
                          b2: Optional[torch.Tensor] = None, lk_c: Optional[torch.Tensor] = None,
                          gen: Optional[GenParams] = None, b_fuse: Optional[torch.Tensor] = None,
                          out: Optional[torch.Tensor] = None, stream=None) -> torch.Tensor:
    """esc_residual_step_forward: f_in + ConvAttn(ConvFFN(f_in), LK) (Eq. 3 line 3)."""
    return _native.residual_step_forward(f_in, w1, k_dw, w2, Ca, lk, w_fuse, workspace, b1, b_dw, b2, lk_c, gen, b_fuse,
                                         out, stream)


def new_dense_workspace(N: int, Ca: int, H: int, W: int, Ks: int, device="cuda", stream=None) -> torch.Tensor:
    """Allocate (with torch) and prepare a workspace for esc_convattn_dense_forward."""
    nbytes = int(load_library().esc_dense_workspace_bytes(N, Ca, H, W, Ks))
    if nbytes == 0:
        raise ValueError("bad shape for a workspace")
    ws = torch.empty(nbytes, dtype=torch.uint8, device=device)
    workspace_init(ws, stream)
    return ws


def convattn_dense_forward(x: torch.Tensor, Ca: int, lk_dense: torch.Tensor, workspace: torch.Tensor,
                           gen: Optional[GenParams] = None, dk_in: Optional[torch.Tensor] = None,
                           out: Optional[torch.Tensor] = None, stream=None) -> torch.Tensor:
    """esc_convattn_dense_forward.  lk_dense is [Ca, Ca, Ks, Ks], output channel first."""
    return _native.convattn_dense_forward(x, Ca, lk_dense, workspace, gen, dk_in, out, stream)


def new_backward_workspace(N: int, Ca: int, H: int, W: int, Ks: int, hidden: int, device="cuda", stream=None) -> torch.Tensor:
    """Allocate (with torch) and prepare a workspace for esc_convattn_backward."""
    nbytes = int(load_library().esc_backward_workspace_bytes(N, Ca, H, W, Ks, hidden))
    if nbytes == 0:
        raise ValueError("bad shape for a workspace")
    ws = torch.empty(nbytes, dtype=torch.uint8, device=device)
    workspace_init(ws, stream)
    return ws


def convattn_backward(x: torch.Tensor, grad_out: torch.Tensor, Ca: int, lk: torch.Tensor, workspace: torch.Tensor,
                      gen: Optional[GenParams] = None, dk_in: Optional[torch.Tensor] = None, accumulate: bool = False,
                      grads: Optional[dict] = None, stream=None) -> dict:
    """esc_convattn_backward.  Returns a dict of device tensors: grad_x, grad_lk, grad_dk and, with an
    estimator, grad_w_up, grad_b_up (and grad_w_down, grad_b_down when hidden > 0).  `grads` may carry
    buffers to write into (required to make sense of accumulate=True)."""
    return _native.convattn_backward(x, grad_out, Ca, lk, workspace, gen, dk_in, accumulate, grads, stream)
