"""ctypes binding of libhydra (the C ABI declared in include/hydra.h).

Argument marshalling only: every step of the path runs in the HIP kernels of
libhydra.  Tensors are PyTorch tensors on a ROCm device (PyTorch provides the
device memory and the stream); they are checked for dtype, shape, device and
contiguity, then their data pointers are passed through.  There is no CPU
fallback: a missing library raises ``HydraLibraryMissing``.

The accepted form of a call goes through ``_hydra_native`` (native/binding.cpp),
which makes the same checks and the same library call without ctypes; for
anything else it answers ``SLOW`` and the Python checks below decide, with
their messages.
"""
from __future__ import annotations

import ctypes
import os
import warnings
from typing import Optional

PKG = os.path.dirname(os.path.abspath(__file__))
LIB_PATH = os.path.join(PKG, "libhydra.so")
NATIVE_PATH = os.path.join(PKG, "_hydra_native.so")

HYDRA_OK = 0
HYDRA_ERR_NULL = -1
HYDRA_ERR_SHAPE = -2
HYDRA_ERR_ALIGN = -3
HYDRA_ERR_UNSUPPORTED = -4
HYDRA_ERR_WORKSPACE = -5
HYDRA_ERR_HIP = -6
HYDRA_MAX_RANK = 128
HYDRA_MAX_GROUP = 8
HYDRA_MAX_ADAPTERS = 4
HYDRA_SCORE_NOALLOC_MAX_BYTES = 48 << 20
HYDRA_GROUP_WS_CONTROL_BYTES = 4352
HYDRA_GROUP_WS_BOUND_WORD = 8
HYDRA_GROUP_WS_T_BYTES = 65536
HYDRA_GROUP_WS_Y_BYTES = 2097152

# Every symbol include/hydra.h declares.
EXPORTED = (
    "hydra_lora_linear",
    "hydra_lora_linear_workspace_bytes",
    "hydra_lora_linear_ws",
    "hydra_lora_linear_group",
    "hydra_lora_linear_group_workspace_bytes",
    "hydra_lora_linear_group_ws",
    "hydra_lora_linear_multi",
    "hydra_lora_linear_multi_workspace_bytes",
    "hydra_lora_linear_multi_ws",
    "hydra_score_workspace_bytes",
    "hydra_score",
    "hydra_score_noalloc",
    "hydra_score_two_input",
    "hydra_score_logits",
    "hydra_value_head",
    "hydra_ppo_advantages",
    "hydra_ppo_loss",
    "hydra_transpose_bf16",
    "hydra_lora_linear_backward_workspace_bytes",
    "hydra_lora_linear_backward",
    "hydra_status_string",
    "hydra_abi_version",
)


class HydraLibraryMissing(ImportError):
    pass


class HydraError(RuntimeError):
    def __init__(self, status: int, where: str):
        self.status = int(status)
        super().__init__(f"{where}: {status_string(status)} ({status})")


_lib: Optional[ctypes.CDLL] = None

_vp = ctypes.c_void_p
_i64 = ctypes.c_int64
_f32 = ctypes.c_float


def lib() -> ctypes.CDLL:
    """Load libhydra.so (built in-tree by ``python -m paper_2309_00754_amd.build``)."""
    global _lib
    if _lib is not None:
        return _lib
    if not os.path.exists(LIB_PATH):
        raise HydraLibraryMissing(
            f"{LIB_PATH} is not built; run `python -m paper_2309_00754_amd.build` (no CPU fallback exists)")
    L = ctypes.CDLL(LIB_PATH)
    L.hydra_lora_linear.argtypes = [_vp, _vp, _vp, _vp, _f32, _i64, _i64, _i64, _i64, _vp, _vp, _vp]
    L.hydra_lora_linear.restype = ctypes.c_int
    _pp = ctypes.POINTER(ctypes.c_void_p)
    L.hydra_lora_linear_group.argtypes = [_i64, _pp, _pp, _pp, _pp, ctypes.POINTER(ctypes.c_float), _i64, _i64, _i64,
                                          _i64, _pp, _pp, _vp]
    L.hydra_lora_linear_group.restype = ctypes.c_int
    L.hydra_lora_linear_group_workspace_bytes.argtypes = [_i64, _i64, _i64, _i64, ctypes.POINTER(ctypes.c_size_t)]
    L.hydra_lora_linear_group_workspace_bytes.restype = ctypes.c_int
    L.hydra_lora_linear_group_ws.argtypes = [_i64, _pp, _pp, _pp, _pp, ctypes.POINTER(ctypes.c_float), _i64, _i64,
                                             _i64, _i64, _pp, _pp, _vp, ctypes.c_size_t, _vp]
    L.hydra_lora_linear_group_ws.restype = ctypes.c_int
    L.hydra_lora_linear_workspace_bytes.argtypes = [_i64, _i64, _i64, ctypes.POINTER(ctypes.c_size_t)]
    L.hydra_lora_linear_workspace_bytes.restype = ctypes.c_int
    L.hydra_lora_linear_ws.argtypes = [_vp, _vp, _vp, _vp, _f32, _i64, _i64, _i64, _i64, _vp, _vp, _vp,
                                       ctypes.c_size_t, _vp]
    L.hydra_lora_linear_ws.restype = ctypes.c_int
    L.hydra_lora_linear_multi.argtypes = [_vp, _vp, _i64, _pp, _pp, _pp, ctypes.POINTER(ctypes.c_float), _i64, _i64,
                                          _i64, _i64, _vp, _pp, _vp]
    L.hydra_lora_linear_multi.restype = ctypes.c_int
    L.hydra_lora_linear_multi_workspace_bytes.argtypes = [_i64, _i64, _i64, ctypes.POINTER(ctypes.c_size_t)]
    L.hydra_lora_linear_multi_workspace_bytes.restype = ctypes.c_int
    L.hydra_lora_linear_multi_ws.argtypes = [_vp, _vp, _i64, _pp, _pp, _pp, ctypes.POINTER(ctypes.c_float), _i64, _i64,
                                             _i64, _i64, _vp, _pp, _vp, ctypes.c_size_t, _vp]
    L.hydra_lora_linear_multi_ws.restype = ctypes.c_int
    L.hydra_score_workspace_bytes.argtypes = [_i64, _i64, ctypes.POINTER(ctypes.c_size_t)]
    L.hydra_score_workspace_bytes.restype = ctypes.c_int
    L.hydra_score.argtypes = [_vp, _vp, _vp, _vp, _f32, _vp, _vp, _i64, _i64, _i64, _i64, _i64,
                              _vp, _vp, _vp, _vp, _vp, _vp, _vp, ctypes.c_size_t, _vp, _vp]
    L.hydra_score.restype = ctypes.c_int
    L.hydra_score_noalloc.argtypes = [_vp, _vp, _vp, _vp, _f32, _vp, _vp, _i64, _i64, _i64, _i64, _i64,
                                      _vp, _vp, _vp, _vp, _vp, _vp, _vp, _vp]
    L.hydra_score_noalloc.restype = ctypes.c_int
    L.hydra_score_two_input.argtypes = [_vp, _vp, _vp, _vp, _vp, _f32, _vp, _vp, _i64, _i64, _i64, _i64, _i64,
                                        _vp, _vp, _vp, _vp, _vp, _vp, _vp, ctypes.c_size_t, _vp, _vp]
    L.hydra_score_two_input.restype = ctypes.c_int
    L.hydra_score_logits.argtypes = [_vp, _vp, _vp, _i64, _i64, _vp, _vp, _vp, _vp, _vp, _vp, _vp]
    L.hydra_score_logits.restype = ctypes.c_int
    L.hydra_value_head.argtypes = [_vp, _vp, _i64, _i64, _vp, _vp]
    L.hydra_value_head.restype = ctypes.c_int
    L.hydra_ppo_advantages.argtypes = [_vp, _vp, _vp, _i64, _i64, _i64, _f32, _f32, _f32, _vp, _vp, _vp, _vp]
    L.hydra_ppo_advantages.restype = ctypes.c_int
    L.hydra_ppo_loss.argtypes = [_vp, _vp, _vp, _vp, _vp, _i64, _i64, _i64, _f32, _vp, _vp, _vp, _vp]
    L.hydra_ppo_loss.restype = ctypes.c_int
    L.hydra_transpose_bf16.argtypes = [_vp, _i64, _i64, _vp, _vp]
    L.hydra_transpose_bf16.restype = ctypes.c_int
    L.hydra_lora_linear_backward_workspace_bytes.argtypes = [_i64, _i64, _i64, _i64, ctypes.POINTER(ctypes.c_size_t)]
    L.hydra_lora_linear_backward_workspace_bytes.restype = ctypes.c_int
    L.hydra_lora_linear_backward.argtypes = [_vp, _vp, _vp, _vp, _f32, _vp, _i64, _i64, _i64, _i64, _vp, _vp, _vp,
                                             _vp, ctypes.c_size_t, _vp]
    L.hydra_lora_linear_backward.restype = ctypes.c_int
    L.hydra_status_string.argtypes = [ctypes.c_int]
    L.hydra_status_string.restype = ctypes.c_char_p
    L.hydra_abi_version.argtypes = []
    L.hydra_abi_version.restype = ctypes.c_int
    _lib = L
    return L


_SLOW = -1000


class _NoNative:
    """Stands in for _hydra_native where it is not built: every call takes the Python path."""

    def __getattr__(self, name):
        return lambda *args: _SLOW


_nat = None


def _native():
    """_hydra_native, loaded with the first call (it needs torch's libraries in the process)."""
    global _nat
    if _nat is None:
        _torch()
        try:
            from . import _hydra_native as nat
        except ImportError as e:
            if os.path.exists(NATIVE_PATH):  # built, and yet not loaded: not to go unnoticed
                warnings.warn(f"{NATIVE_PATH} does not load, calls go through ctypes and take longer on the host: "
                              f"{e}", RuntimeWarning, stacklevel=3)
            nat = _NoNative()
        _nat = nat
    return _nat


def status_string(status: int) -> str:
    return lib().hydra_status_string(int(status)).decode()


def _check(status: int, where: str) -> None:
    if status != HYDRA_OK:
        raise HydraError(status, where)


# ------------------------------------------------------------------ tensor helpers

def _torch():
    import torch
    return torch


def _ptr(t) -> Optional[int]:
    return None if t is None else int(t.data_ptr())


def _stream_handle(stream) -> Optional[int]:
    """The hipStream_t of ``stream``, or of torch's current stream on the current device when None (read through
    torch's raw-stream query when it has one: building a Stream object costs a few microseconds per call)."""
    torch = _torch()
    if stream is None:
        raw = getattr(torch._C, "_cuda_getCurrentRawStream", None)
        if raw is not None:
            return int(raw(torch.cuda.current_device()))
        stream = torch.cuda.current_stream()
    return int(stream.cuda_stream)


def _need(t, name, dtypes, shape=None):
    if t is None:
        return
    torch = _torch()
    # the accepted case in one condition (a few attribute reads: these checks run for every tensor of every call,
    # and at decode sizes the host time of a call is comparable to its kernel's); the messages only on failure
    if isinstance(t, torch.Tensor) and t.is_cuda and t.dtype in dtypes and t.is_contiguous() and (
            shape is None or t.shape == tuple(shape)):
        return
    if not isinstance(t, torch.Tensor):
        raise TypeError(f"{name} must be a torch.Tensor")
    if t.device.type != "cuda":
        raise ValueError(f"{name} must be on a ROCm device, got {t.device}")
    if t.dtype not in dtypes:
        raise TypeError(f"{name} has dtype {t.dtype}, expected one of {dtypes}")
    if not t.is_contiguous():
        raise ValueError(f"{name} must be contiguous")
    if shape is not None and tuple(t.shape) != tuple(shape):
        raise ValueError(f"{name} has shape {tuple(t.shape)}, expected {tuple(shape)}")


def _bf16_types():
    torch = _torch()
    return (torch.bfloat16, torch.int16, torch.uint16)


# ------------------------------------------------------------------ entry points

def hydra_lora_linear(x, W, A, B, s: float, y_off=None, y_on=None, stream=None) -> None:
    """y_off = x W^T and/or y_on = x W^T + s (x A^T) B^T (see include/hydra.h).

    x [M,K], W [N,K], A [r,K], B [N,r]: bf16 (or 16-bit integer tensors holding
    bf16 bits); y_off, y_on [M,N] float32 outputs (either may be None).
    """
    st = (_nat or _native()).lora_linear(x, W, A, B, s, y_off, y_on, None, stream, False)
    if st == _SLOW:
        return _hydra_lora_linear(x, W, A, B, s, y_off, y_on, stream)
    if st != HYDRA_OK:
        _check(st, "hydra_lora_linear")


def _hydra_lora_linear(x, W, A, B, s, y_off, y_on, stream) -> None:
    torch = _torch()
    bf = _bf16_types()
    M, K = x.shape
    N = W.shape[0]
    r = 0 if A is None else A.shape[0]
    _need(x, "x", bf)
    _need(W, "W", bf, (N, K))
    _need(A, "A", bf, (r, K))
    _need(B, "B", bf, (N, r))
    _need(y_off, "y_off", (torch.float32,), (M, N))
    _need(y_on, "y_on", (torch.float32,), (M, N))
    st = lib().hydra_lora_linear(_ptr(x), _ptr(W), _ptr(A), _ptr(B), float(s), M, N, K, r,
                                 _ptr(y_off), _ptr(y_on), _stream_handle(stream))
    _check(st, "hydra_lora_linear")


def hydra_lora_linear_workspace_bytes(M: int, N: int, r: int) -> int:
    out = ctypes.c_size_t(0)
    _check(lib().hydra_lora_linear_workspace_bytes(int(M), int(N), int(r), ctypes.byref(out)),
           "hydra_lora_linear_workspace_bytes")
    return int(out.value)


def hydra_lora_linear_ws(x, W, A, B, s: float, y_off=None, y_on=None, workspace=None, stream=None) -> None:
    """hydra_lora_linear with the pre-pass workspace (see include/hydra.h); allocates one if none is given."""
    st = (_nat or _native()).lora_linear(x, W, A, B, s, y_off, y_on, workspace, stream, True)
    if st == _SLOW:
        return _hydra_lora_linear_ws(x, W, A, B, s, y_off, y_on, workspace, stream)
    if st != HYDRA_OK:
        _check(st, "hydra_lora_linear_ws")


def _hydra_lora_linear_ws(x, W, A, B, s, y_off, y_on, workspace, stream) -> None:
    torch = _torch()
    bf = _bf16_types()
    M, K = x.shape
    N = W.shape[0]
    r = 0 if A is None else A.shape[0]
    _need(x, "x", bf)
    _need(W, "W", bf, (N, K))
    _need(A, "A", bf, (r, K))
    _need(B, "B", bf, (N, r))
    _need(y_off, "y_off", (torch.float32,), (M, N))
    _need(y_on, "y_on", (torch.float32,), (M, N))
    need = hydra_lora_linear_workspace_bytes(M, N, r)
    if workspace is None and need > 0:
        workspace = torch.empty(need, dtype=torch.uint8, device=x.device)
    _need(workspace, "workspace", (torch.uint8,))
    nbytes = 0 if workspace is None else workspace.numel()
    st = lib().hydra_lora_linear_ws(_ptr(x), _ptr(W), _ptr(A), _ptr(B), float(s), M, N, K, r, _ptr(y_off),
                                    _ptr(y_on), _ptr(workspace), nbytes, _stream_handle(stream))
    _check(st, "hydra_lora_linear_ws")


def _ptr_array(ts):
    arr = (ctypes.c_void_p * len(ts))()
    for i, t in enumerate(ts):
        arr[i] = _ptr(t)
    return arr


def hydra_lora_linear_group(xs, Ws, As, Bs, ss, y_offs=None, y_ons=None, stream=None) -> None:
    """G linears with shared M, N, K, r in one call (see include/hydra.h).

    xs, Ws, As, Bs, y_offs, y_ons: sequences of G tensors (entries may be None);
    ss: G scales.
    """
    st = (_nat or _native()).lora_linear_group(xs, Ws, As, Bs, ss, y_offs, y_ons, None, stream, False)
    if st == _SLOW:
        return _hydra_lora_linear_group(xs, Ws, As, Bs, ss, y_offs, y_ons, stream)
    if st != HYDRA_OK:
        _check(st, "hydra_lora_linear_group")


def _hydra_lora_linear_group(xs, Ws, As, Bs, ss, y_offs, y_ons, stream) -> None:
    torch = _torch()
    bf = _bf16_types()
    G = len(Ws)
    if not (len(xs) == len(As) == len(Bs) == len(ss) == G):
        raise ValueError("all per-member sequences must have the same length")
    y_offs = list(y_offs) if y_offs is not None else [None] * G
    y_ons = list(y_ons) if y_ons is not None else [None] * G
    M, K = xs[0].shape
    N = Ws[0].shape[0]
    r = next((a.shape[0] for a in As if a is not None), 0)
    for i in range(G):
        _need(xs[i], "x", bf, (M, K))
        _need(Ws[i], "W", bf, (N, K))
        _need(As[i], "A", bf, (r, K))
        _need(Bs[i], "B", bf, (N, r))
        _need(y_offs[i], "y_off", (torch.float32,), (M, N))
        _need(y_ons[i], "y_on", (torch.float32,), (M, N))
    svals = (ctypes.c_float * G)(*[float(v) for v in ss])
    st = lib().hydra_lora_linear_group(G, _ptr_array(xs), _ptr_array(Ws), _ptr_array(As), _ptr_array(Bs), svals,
                                       M, N, K, r, _ptr_array(y_offs), _ptr_array(y_ons), _stream_handle(stream))
    _check(st, "hydra_lora_linear_group")


def hydra_lora_linear_group_workspace_bytes(G: int, M: int, N: int, r: int) -> int:
    out = ctypes.c_size_t(0)
    _check(lib().hydra_lora_linear_group_workspace_bytes(int(G), int(M), int(N), int(r), ctypes.byref(out)),
           "hydra_lora_linear_group_workspace_bytes")
    return int(out.value)


def hydra_lora_linear_group_workspace(G: int, M: int, N: int, r: int, device):
    """A zero-filled workspace for hydra_lora_linear_group_ws (the calls leave its control words zero, so it is
    reused as it is)."""
    torch = _torch()
    return torch.zeros(hydra_lora_linear_group_workspace_bytes(G, M, N, r), dtype=torch.uint8, device=device)


def hydra_lora_linear_group_ws(xs, Ws, As, Bs, ss, y_offs=None, y_ons=None, workspace=None, stream=None) -> None:
    """hydra_lora_linear_group with a caller workspace: a decode step (M <= 8) in one launch (see include/hydra.h).

    workspace: a uint8 tensor from hydra_lora_linear_group_workspace (zero before its first use)."""
    st = (_nat or _native()).lora_linear_group(xs, Ws, As, Bs, ss, y_offs, y_ons, workspace, stream, True)
    if st == _SLOW:
        return _hydra_lora_linear_group_ws(xs, Ws, As, Bs, ss, y_offs, y_ons, workspace, stream)
    if st != HYDRA_OK:
        _check(st, "hydra_lora_linear_group_ws")


def _hydra_lora_linear_group_ws(xs, Ws, As, Bs, ss, y_offs, y_ons, workspace, stream) -> None:
    torch = _torch()
    bf = _bf16_types()
    G = len(Ws)
    if not (len(xs) == len(As) == len(Bs) == len(ss) == G):
        raise ValueError("all per-member sequences must have the same length")
    y_offs = list(y_offs) if y_offs is not None else [None] * G
    y_ons = list(y_ons) if y_ons is not None else [None] * G
    M, K = xs[0].shape
    N = Ws[0].shape[0]
    r = next((a.shape[0] for a in As if a is not None), 0)
    for i in range(G):
        _need(xs[i], "x", bf, (M, K))
        _need(Ws[i], "W", bf, (N, K))
        _need(As[i], "A", bf, (r, K))
        _need(Bs[i], "B", bf, (N, r))
        _need(y_offs[i], "y_off", (torch.float32,), (M, N))
        _need(y_ons[i], "y_on", (torch.float32,), (M, N))
    if workspace is None:
        raise ValueError("hydra_lora_linear_group_ws needs a workspace from hydra_lora_linear_group_workspace")
    _need(workspace, "workspace", (torch.uint8,))
    svals = (ctypes.c_float * G)(*[float(v) for v in ss])
    st = lib().hydra_lora_linear_group_ws(G, _ptr_array(xs), _ptr_array(Ws), _ptr_array(As), _ptr_array(Bs), svals,
                                          M, N, K, r, _ptr_array(y_offs), _ptr_array(y_ons), _ptr(workspace),
                                          workspace.numel(), _stream_handle(stream))
    _check(st, "hydra_lora_linear_group_ws")


def _multi_args(x_off, W, x_ons, As, Bs, ss, y_off, y_ons):
    torch = _torch()
    bf = _bf16_types()
    n_on = len(x_ons)
    As = list(As) if As is not None else [None] * n_on
    Bs = list(Bs) if Bs is not None else [None] * n_on
    y_ons = list(y_ons) if y_ons is not None else [None] * n_on
    if not (len(As) == len(Bs) == len(ss) == len(y_ons) == n_on):
        raise ValueError("all per-input sequences must have the same length")
    ref = x_off if x_off is not None else (x_ons[0] if n_on else None)
    if ref is None:
        raise ValueError("at least one input is needed")
    M, K = ref.shape
    N = W.shape[0]
    r = next((a.shape[0] for a in As if a is not None), 0)
    _need(W, "W", bf, (N, K))
    _need(x_off, "x_off", bf, (M, K))
    _need(y_off, "y_off", (torch.float32,), (M, N))
    for a in range(n_on):
        _need(x_ons[a], "x_on", bf, (M, K))
        _need(As[a], "A", bf, (r, K))
        _need(Bs[a], "B", bf, (N, r))
        _need(y_ons[a], "y_on", (torch.float32,), (M, N))
    svals = (ctypes.c_float * max(n_on, 1))(*[float(v) for v in ss])
    return (_ptr(x_off), _ptr(W), n_on, _ptr_array(x_ons), _ptr_array(As), _ptr_array(Bs), svals if n_on else None, M,
            N, K, r, _ptr(y_off), _ptr_array(y_ons))


def hydra_lora_linear_multi(x_off, W, x_ons, As, Bs, ss, y_off=None, y_ons=None, stream=None) -> None:
    """One W for a LoRA-off input and several LoRA-on inputs with their own adapters (see include/hydra.h).

    x_off, y_off: tensors or None (together); x_ons, As, Bs, y_ons: sequences of n_on tensors (As, Bs may be
    None or all-None when r == 0); ss: n_on scales.
    """
    st = (_nat or _native()).lora_linear_multi(x_off, W, x_ons, As, Bs, ss, y_off, y_ons, None, stream, False)
    if st == _SLOW:
        return _hydra_lora_linear_multi(x_off, W, x_ons, As, Bs, ss, y_off, y_ons, stream)
    if st != HYDRA_OK:
        _check(st, "hydra_lora_linear_multi")


def _hydra_lora_linear_multi(x_off, W, x_ons, As, Bs, ss, y_off, y_ons, stream) -> None:
    st = lib().hydra_lora_linear_multi(*_multi_args(x_off, W, x_ons, As, Bs, ss, y_off, y_ons), _stream_handle(stream))
    _check(st, "hydra_lora_linear_multi")


def hydra_lora_linear_multi_workspace_bytes(M: int, N: int, r: int) -> int:
    out = ctypes.c_size_t(0)
    _check(lib().hydra_lora_linear_multi_workspace_bytes(int(M), int(N), int(r), ctypes.byref(out)),
           "hydra_lora_linear_multi_workspace_bytes")
    return int(out.value)


def hydra_lora_linear_multi_ws(x_off, W, x_ons, As, Bs, ss, y_off=None, y_ons=None, workspace=None,
                               stream=None) -> None:
    """hydra_lora_linear_multi with a caller workspace (rank 128 at every M; see include/hydra.h).

    workspace: a uint8 tensor of at least hydra_lora_linear_multi_workspace_bytes(M, N, r) bytes."""
    st = (_nat or _native()).lora_linear_multi(x_off, W, x_ons, As, Bs, ss, y_off, y_ons, workspace, stream, True)
    if st == _SLOW:
        return _hydra_lora_linear_multi_ws(x_off, W, x_ons, As, Bs, ss, y_off, y_ons, workspace, stream)
    if st != HYDRA_OK:
        _check(st, "hydra_lora_linear_multi_ws")


def _hydra_lora_linear_multi_ws(x_off, W, x_ons, As, Bs, ss, y_off, y_ons, workspace, stream) -> None:
    torch = _torch()
    if workspace is None:
        raise ValueError("hydra_lora_linear_multi_ws needs a workspace")
    _need(workspace, "workspace", (torch.uint8,))
    st = lib().hydra_lora_linear_multi_ws(*_multi_args(x_off, W, x_ons, As, Bs, ss, y_off, y_ons), _ptr(workspace),
                                          workspace.numel(), _stream_handle(stream))
    _check(st, "hydra_lora_linear_multi_ws")


def hydra_score_workspace_bytes(M: int, V: int) -> int:
    out = ctypes.c_size_t(0)
    _check(lib().hydra_score_workspace_bytes(int(M), int(V), ctypes.byref(out)), "hydra_score_workspace_bytes")
    return int(out.value)


def hydra_score(h, W_lm, A, B, s: float, tokens, w_rm, n_seq: int, seq_len: int,
                lp_on, lp_off, kl, reward=None, lse_on=None, lse_off=None,
                workspace=None, err_flag=None, stream=None) -> None:
    """Fused CLM-head (LoRA on and off) log-prob / KL scoring plus the reward head."""
    st = (_nat or _native()).score(None, h, W_lm, A, B, s, tokens, w_rm, n_seq, seq_len, lp_on, lp_off, kl, reward,
                                   lse_on, lse_off, workspace, err_flag, stream, False)
    if st == _SLOW:
        return _hydra_score(h, W_lm, A, B, s, tokens, w_rm, n_seq, seq_len, lp_on, lp_off, kl, reward, lse_on,
                            lse_off, workspace, err_flag, stream)
    if st != HYDRA_OK:
        _check(st, "hydra_score")


def _hydra_score(h, W_lm, A, B, s, tokens, w_rm, n_seq, seq_len, lp_on, lp_off, kl, reward, lse_on, lse_off,
                 workspace, err_flag, stream) -> None:
    torch = _torch()
    bf = _bf16_types()
    M, K = h.shape
    V = W_lm.shape[0]
    r = 0 if A is None else A.shape[0]
    if M != n_seq * seq_len:
        raise ValueError("h rows must equal n_seq * seq_len")
    _need(h, "h", bf)
    _need(W_lm, "W_lm", bf, (V, K))
    _need(A, "A", bf, (r, K))
    _need(B, "B", bf, (V, r))
    _need(tokens, "tokens", (torch.int32,), (M,))
    _need(w_rm, "w_rm", bf, (K,))
    for name, t in (("lp_on", lp_on), ("lp_off", lp_off), ("kl", kl), ("lse_on", lse_on), ("lse_off", lse_off)):
        _need(t, name, (torch.float32,), (M,))
    _need(reward, "reward", (torch.float32,), (n_seq,))
    _need(err_flag, "err_flag", (torch.int32,), (1,))
    need = hydra_score_workspace_bytes(M, V)
    if workspace is None:
        workspace = torch.empty(need, dtype=torch.uint8, device=h.device)
    _need(workspace, "workspace", (torch.uint8,))
    st = lib().hydra_score(_ptr(h), _ptr(W_lm), _ptr(A), _ptr(B), float(s), _ptr(tokens), _ptr(w_rm),
                           int(n_seq), int(seq_len), K, V, r, _ptr(lp_on), _ptr(lp_off), _ptr(kl), _ptr(reward),
                           _ptr(lse_on), _ptr(lse_off), _ptr(workspace), workspace.numel(), _ptr(err_flag),
                           _stream_handle(stream))
    _check(st, "hydra_score")


def hydra_score_two_input(h_act, h_off, W_lm, A, B, s: float, tokens, w_rm, n_seq: int, seq_len: int,
                          lp_on, lp_off, kl, reward=None, lse_on=None, lse_off=None,
                          workspace=None, err_flag=None, stream=None) -> None:
    """Scoring with the actor pass's own hidden states (h_act, with the head's LoRA) and the LoRA-off pass's (h_off:
    reference log-probabilities and reward), one launch over both (see include/hydra.h)."""
    st = (_nat or _native()).score(h_act, h_off, W_lm, A, B, s, tokens, w_rm, n_seq, seq_len, lp_on, lp_off, kl,
                                   reward,
                                   lse_on, lse_off, workspace, err_flag, stream, False) if h_act is not None else _SLOW
    if st == _SLOW:
        return _hydra_score_two_input(h_act, h_off, W_lm, A, B, s, tokens, w_rm, n_seq, seq_len, lp_on, lp_off, kl,
                                      reward, lse_on, lse_off, workspace, err_flag, stream)
    if st != HYDRA_OK:
        _check(st, "hydra_score_two_input")


def _hydra_score_two_input(h_act, h_off, W_lm, A, B, s, tokens, w_rm, n_seq, seq_len, lp_on, lp_off, kl, reward,
                           lse_on, lse_off, workspace, err_flag, stream) -> None:
    torch = _torch()
    bf = _bf16_types()
    M, K = h_off.shape
    V = W_lm.shape[0]
    r = 0 if A is None else A.shape[0]
    if M != n_seq * seq_len:
        raise ValueError("h rows must equal n_seq * seq_len")
    _need(h_act, "h_act", bf, (M, K))
    _need(h_off, "h_off", bf, (M, K))
    _need(W_lm, "W_lm", bf, (V, K))
    _need(A, "A", bf, (r, K))
    _need(B, "B", bf, (V, r))
    _need(tokens, "tokens", (torch.int32,), (M,))
    _need(w_rm, "w_rm", bf, (K,))
    for name, t in (("lp_on", lp_on), ("lp_off", lp_off), ("kl", kl), ("lse_on", lse_on), ("lse_off", lse_off)):
        _need(t, name, (torch.float32,), (M,))
    _need(reward, "reward", (torch.float32,), (n_seq,))
    _need(err_flag, "err_flag", (torch.int32,), (1,))
    if workspace is None:
        workspace = torch.empty(hydra_score_workspace_bytes(M, V), dtype=torch.uint8, device=h_off.device)
    _need(workspace, "workspace", (torch.uint8,))
    st = lib().hydra_score_two_input(_ptr(h_act), _ptr(h_off), _ptr(W_lm), _ptr(A), _ptr(B), float(s), _ptr(tokens),
                                     _ptr(w_rm), int(n_seq), int(seq_len), K, V, r, _ptr(lp_on), _ptr(lp_off),
                                     _ptr(kl), _ptr(reward), _ptr(lse_on), _ptr(lse_off), _ptr(workspace),
                                     workspace.numel(), _ptr(err_flag), _stream_handle(stream))
    _check(st, "hydra_score_two_input")


def hydra_score_noalloc(h, W_lm, A, B, s: float, tokens, w_rm, n_seq: int, seq_len: int,
                        lp_on, lp_off, kl, reward=None, lse_on=None, lse_off=None, err_flag=None,
                        stream=None) -> None:
    """hydra_score with its workspace in the library's own device scratch (no allocation by the call)."""
    st = (_nat or _native()).score(None, h, W_lm, A, B, s, tokens, w_rm, n_seq, seq_len, lp_on, lp_off, kl, reward,
                                   lse_on, lse_off, None, err_flag, stream, True)
    if st == _SLOW:
        return _hydra_score_noalloc(h, W_lm, A, B, s, tokens, w_rm, n_seq, seq_len, lp_on, lp_off, kl, reward, lse_on,
                                    lse_off, err_flag, stream)
    if st != HYDRA_OK:
        _check(st, "hydra_score_noalloc")


def _hydra_score_noalloc(h, W_lm, A, B, s, tokens, w_rm, n_seq, seq_len, lp_on, lp_off, kl, reward, lse_on, lse_off,
                         err_flag, stream) -> None:
    torch = _torch()
    bf = _bf16_types()
    M, K = h.shape
    V = W_lm.shape[0]
    r = 0 if A is None else A.shape[0]
    if M != n_seq * seq_len:
        raise ValueError("h rows must equal n_seq * seq_len")
    _need(h, "h", bf)
    _need(W_lm, "W_lm", bf, (V, K))
    _need(A, "A", bf, (r, K))
    _need(B, "B", bf, (V, r))
    _need(tokens, "tokens", (torch.int32,), (M,))
    _need(w_rm, "w_rm", bf, (K,))
    for name, t in (("lp_on", lp_on), ("lp_off", lp_off), ("kl", kl), ("lse_on", lse_on), ("lse_off", lse_off)):
        _need(t, name, (torch.float32,), (M,))
    _need(reward, "reward", (torch.float32,), (n_seq,))
    _need(err_flag, "err_flag", (torch.int32,), (1,))
    st = lib().hydra_score_noalloc(_ptr(h), _ptr(W_lm), _ptr(A), _ptr(B), float(s), _ptr(tokens), _ptr(w_rm),
                                   int(n_seq), int(seq_len), K, V, r, _ptr(lp_on), _ptr(lp_off), _ptr(kl),
                                   _ptr(reward), _ptr(lse_on), _ptr(lse_off), _ptr(err_flag), _stream_handle(stream))
    _check(st, "hydra_score_noalloc")


def hydra_score_logits(logits_on, logits_off, tokens, lp_on, lp_off, kl,
                       lse_on=None, lse_off=None, err_flag=None, stream=None) -> None:
    """Sampled-token log-probabilities and KL from materialised fp32 logits."""
    st = (_nat or _native()).score_logits(logits_on, logits_off, tokens, lp_on, lp_off, kl, lse_on, lse_off, err_flag,
                                          stream)
    if st == _SLOW:
        return _hydra_score_logits(logits_on, logits_off, tokens, lp_on, lp_off, kl, lse_on, lse_off, err_flag,
                                   stream)
    if st != HYDRA_OK:
        _check(st, "hydra_score_logits")


def _hydra_score_logits(logits_on, logits_off, tokens, lp_on, lp_off, kl, lse_on, lse_off, err_flag, stream) -> None:
    torch = _torch()
    M, V = logits_on.shape
    _need(logits_on, "logits_on", (torch.float32,))
    _need(logits_off, "logits_off", (torch.float32,), (M, V))
    _need(tokens, "tokens", (torch.int32,), (M,))
    for name, t in (("lp_on", lp_on), ("lp_off", lp_off), ("kl", kl), ("lse_on", lse_on), ("lse_off", lse_off)):
        _need(t, name, (torch.float32,), (M,))
    _need(err_flag, "err_flag", (torch.int32,), (1,))
    st = lib().hydra_score_logits(_ptr(logits_on), _ptr(logits_off), _ptr(tokens), M, V, _ptr(lp_on), _ptr(lp_off),
                                  _ptr(kl), _ptr(lse_on), _ptr(lse_off), _ptr(err_flag), _stream_handle(stream))
    _check(st, "hydra_score_logits")


def hydra_value_head(h, w_v, values, stream=None) -> None:
    """values[m] = <h[m], w_v>: the critic's scalar head on every row (see include/hydra.h)."""
    st = (_nat or _native()).value_head(h, w_v, values, stream)
    if st == _SLOW:
        return _hydra_value_head(h, w_v, values, stream)
    if st != HYDRA_OK:
        _check(st, "hydra_value_head")


def _hydra_value_head(h, w_v, values, stream) -> None:
    torch = _torch()
    bf = _bf16_types()
    M, K = h.shape
    _need(h, "h", bf)
    _need(w_v, "w_v", bf, (K,))
    _need(values, "values", (torch.float32,), (M,))
    st = lib().hydra_value_head(_ptr(h), _ptr(w_v), M, K, _ptr(values), _stream_handle(stream))
    _check(st, "hydra_value_head")


def hydra_ppo_advantages(kl, reward, values, n_seq: int, seq_len: int, advantages, returns, rewards=None,
                         start: int = 0, beta: float = 0.02, gamma: float = 1.0, lam: float = 0.95,
                         stream=None) -> None:
    """Per-token PPO reward and GAE advantages / returns (see include/hydra.h)."""
    st = (_nat or _native()).ppo_advantages(kl, reward, values, n_seq, seq_len, start, beta, gamma, lam, rewards,
                                            advantages, returns, stream)
    if st == _SLOW:
        return _hydra_ppo_advantages(kl, reward, values, n_seq, seq_len, advantages, returns, rewards, start, beta,
                                     gamma, lam, stream)
    if st != HYDRA_OK:
        _check(st, "hydra_ppo_advantages")


def _hydra_ppo_advantages(kl, reward, values, n_seq, seq_len, advantages, returns, rewards, start, beta, gamma, lam,
                          stream) -> None:
    torch = _torch()
    M = int(n_seq) * int(seq_len)
    for name, t, n in (("kl", kl, M), ("reward", reward, n_seq), ("values", values, M), ("advantages", advantages, M),
                       ("returns", returns, M), ("rewards", rewards, M)):
        _need(t, name, (torch.float32,), (n,))
    st = lib().hydra_ppo_advantages(_ptr(kl), _ptr(reward), _ptr(values), int(n_seq), int(seq_len), int(start),
                                    float(beta), float(gamma), float(lam), _ptr(rewards), _ptr(advantages),
                                    _ptr(returns), _stream_handle(stream))
    _check(st, "hydra_ppo_advantages")


def hydra_ppo_loss(lp_new, lp_old, advantages, values, returns, n_seq: int, seq_len: int, losses, d_lp=None,
                   d_v=None, start: int = 0, eps: float = 0.2, stream=None) -> None:
    """PPO policy and value losses with their per-token gradients (see include/hydra.h)."""
    st = (_nat or _native()).ppo_loss(lp_new, lp_old, advantages, values, returns, n_seq, seq_len, start, eps, losses,
                                      d_lp, d_v, stream)
    if st == _SLOW:
        return _hydra_ppo_loss(lp_new, lp_old, advantages, values, returns, n_seq, seq_len, losses, d_lp, d_v, start,
                               eps, stream)
    if st != HYDRA_OK:
        _check(st, "hydra_ppo_loss")


def _hydra_ppo_loss(lp_new, lp_old, advantages, values, returns, n_seq, seq_len, losses, d_lp, d_v, start, eps,
                    stream) -> None:
    torch = _torch()
    M = int(n_seq) * int(seq_len)
    for t, name in ((lp_new, "lp_new"), (lp_old, "lp_old"), (advantages, "advantages"), (values, "values"),
                    (returns, "returns"), (d_lp, "d_lp"), (d_v, "d_v")):
        _need(t, name, (torch.float32,), (M,))
    _need(losses, "losses", (torch.float32,), (3,))
    st = lib().hydra_ppo_loss(_ptr(lp_new), _ptr(lp_old), _ptr(advantages), _ptr(values), _ptr(returns),
                              int(n_seq), int(seq_len), int(start), float(eps), _ptr(losses), _ptr(d_lp),
                              _ptr(d_v), _stream_handle(stream))
    _check(st, "hydra_ppo_loss")


def hydra_transpose_bf16(src, dst, stream=None) -> None:
    """dst [C,R] = src [R,C]^T for 16-bit tensors (see include/hydra.h)."""
    bf = _bf16_types()
    R, C = src.shape
    _need(src, "src", bf)
    _need(dst, "dst", bf, (C, R))
    _check(lib().hydra_transpose_bf16(_ptr(src), R, C, _ptr(dst), _stream_handle(stream)), "hydra_transpose_bf16")


def hydra_lora_linear_backward_workspace_bytes(M: int, N: int, K: int, r: int) -> int:
    out = ctypes.c_size_t(0)
    _check(lib().hydra_lora_linear_backward_workspace_bytes(int(M), int(N), int(K), int(r), ctypes.byref(out)),
           "hydra_lora_linear_backward_workspace_bytes")
    return int(out.value)


def hydra_lora_linear_backward(x, Wt, A, B, s: float, dy, dx=None, dA=None, dB=None, workspace=None,
                               stream=None) -> None:
    """dx, dA, dB of y = x W^T + s (x A^T) B^T with W frozen (see include/hydra.h).

    x [M,K], Wt [K,N] (W transposed, may be None when dx is not wanted), A [r,K],
    B [N,r], dy [M,N]: bf16 (or 16-bit integer tensors holding bf16 bits);
    dx [M,K], dA [r,K], dB [N,r] float32 outputs (each optional).  Allocates
    the workspace if none is given.
    """
    st = (_nat or _native()).lora_linear_backward(x, Wt, A, B, s, dy, dx, dA, dB, workspace, stream)
    if st == _SLOW:
        return _hydra_lora_linear_backward(x, Wt, A, B, s, dy, dx, dA, dB, workspace, stream)
    if st != HYDRA_OK:
        _check(st, "hydra_lora_linear_backward")


def _hydra_lora_linear_backward(x, Wt, A, B, s, dy, dx, dA, dB, workspace, stream) -> None:
    torch = _torch()
    bf = _bf16_types()
    M, N = dy.shape
    K = A.shape[1] if A is not None else (x.shape[1] if x is not None else Wt.shape[0])
    r = 0 if A is None else A.shape[0]
    _need(x, "x", bf, (M, K))
    _need(Wt, "Wt", bf, (K, N))
    _need(A, "A", bf, (r, K))
    _need(B, "B", bf, (N, r))
    _need(dy, "dy", bf)
    _need(dx, "dx", (torch.float32,), (M, K))
    _need(dA, "dA", (torch.float32,), (r, K))
    _need(dB, "dB", (torch.float32,), (N, r))
    need = hydra_lora_linear_backward_workspace_bytes(M, N, K, r)
    if workspace is None and need > 0:
        workspace = torch.empty(need, dtype=torch.uint8, device=dy.device)
    _need(workspace, "workspace", (torch.uint8,))
    nbytes = 0 if workspace is None else workspace.numel()
    st = lib().hydra_lora_linear_backward(_ptr(x), _ptr(Wt), _ptr(A), _ptr(B), float(s), _ptr(dy), M, N, K, r,
                                          _ptr(dx), _ptr(dA), _ptr(dB), _ptr(workspace), nbytes,
                                          _stream_handle(stream))
    _check(st, "hydra_lora_linear_backward")
