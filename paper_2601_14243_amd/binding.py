"""Binding of libjet.so: argument marshalling only.

``jet_*`` functions mirror include/jet.h one to one through ctypes (raw pointers, sizes, a
stream handle; they return the status code).  The un-prefixed helpers take
torch CUDA tensors, allocate the outputs with torch, pass ``data_ptr()`` and the
current stream, and raise ``JetError`` on a non-zero status.  Calls of the plain form (exact tensors of
the right type and shape) are answered by the extension ``_jet_host`` (csrc/jet_host.cpp), which does the
same in one native call; what it does not take (None) goes through the Python code here, which also words
the errors and takes every call, with a warning, where the extension is missing or was built for another Python or
torch.  No arithmetic of the method happens in Python, and libjet.so has no fallback: if it is missing the first
call fails loudly.
"""
from __future__ import annotations

import ctypes
import importlib
import os
import warnings

import torch

_HERE = os.path.dirname(os.path.abspath(__file__))
_LIB_PATH = os.path.join(_HERE, "libjet.so")

JET_SRC_BF16 = 0
JET_SRC_FP8_ROW = 1
GROUP = 128

_HOST_PATH = os.path.join(_HERE, "_jet_host.so")

_lib = None
_host = None


class JetError(RuntimeError):
    def __init__(self, status: int, where: str):
        self.status = status
        super().__init__(f"{where}: jet_status {status} ({jet_status_str(status)})")


def lib() -> ctypes.CDLL:
    """Load libjet.so (built in-tree by paper_2601_14243_amd.build)."""
    global _lib
    if _lib is None:
        if not os.path.exists(_LIB_PATH):
            raise FileNotFoundError(
                f"{_LIB_PATH} is missing: build it with `python -m paper_2601_14243_amd.build` "
                "(there is no CPU or PyTorch fallback)")
        L = ctypes.CDLL(_LIB_PATH)
        vp, i64, i32 = ctypes.c_void_p, ctypes.c_int64, ctypes.c_int
        L.jet_quant_act.restype = i32
        L.jet_quant_act.argtypes = [vp, vp, i32, i64, i64, vp, vp, vp, vp, vp]
        L.jet_quant_weight.restype = i32
        L.jet_quant_weight.argtypes = [vp, i64, i64, vp, vp, vp, vp, vp]
        for name in ("jet_fp8_linear_fwd", "jet_fp8_linear_dgrad", "jet_fp8_linear_wgrad"):
            f = getattr(L, name)
            f.restype = i32
            f.argtypes = [vp, vp, vp, vp, vp, i64, i64, i64, vp]
        L.jet_rmsnorm_quant.restype = i32
        L.jet_rmsnorm_quant.argtypes = [vp, vp, ctypes.c_float, i64, i64, vp, vp, vp]
        L.jet_silu_mul_quant.restype = i32
        L.jet_silu_mul_quant.argtypes = [vp, vp, i64, i64, i64, vp, vp, vp]
        L.jet_silu_mul_bwd_quant.restype = i32
        L.jet_silu_mul_bwd_quant.argtypes = [vp, vp, i64, vp, i64, i64, vp, vp, vp, vp, vp, vp]
        L.jet_silu_mul_bwd.restype = i32
        L.jet_silu_mul_bwd.argtypes = [vp, vp, i64, vp, i64, i64, vp, vp, i64, vp]
        L.jet_status_str.restype = ctypes.c_char_p
        L.jet_status_str.argtypes = [i32]
        L.jet_version.restype = i32
        _lib = L
    return _lib


class _PythonMarshalling:
    """Stands in for the extension where it cannot be loaded: takes no call, so that the Python code does."""

    @staticmethod
    def _declined(*args):
        return None

    quant_act = rmsnorm_quant = silu_mul_quant = silu_mul_bwd = quant_weight = gemm = _declined


def _native():
    """Load the native marshalling (built in-tree beside libjet.so)."""
    global _host
    if _host is None:
        lib()
        try:
            if not os.path.exists(_HOST_PATH):
                raise ImportError(f"{_HOST_PATH} is missing")
            host = importlib.import_module("._jet_host", __package__)
            host.init(JetError, getattr(torch, "OutOfMemoryError", torch.cuda.OutOfMemoryError))
        except ImportError as e:
            warnings.warn(f"native marshalling not available ({e}); build it with `python -m paper_2601_14243_amd.build`.  "
                          "The kernels are the same, a call takes some 5 us more on the host.", RuntimeWarning, stacklevel=3)
            host = _PythonMarshalling
        _host = host
    return _host


# ---------------------------------------------------------------- raw calls

def jet_version() -> int:
    return int(lib().jet_version())


def jet_status_str(status: int) -> str:
    return lib().jet_status_str(int(status)).decode()


def jet_quant_act(x, x_scales, src, M, K, q_row, s_row, q_colT, s_colT, stream) -> int:
    return int(lib().jet_quant_act(x, x_scales, src, M, K, q_row, s_row, q_colT, s_colT, stream))


def jet_quant_weight(w, N, K, q, s, qT, sT, stream) -> int:
    return int(lib().jet_quant_weight(w, N, K, q, s, qT, sT, stream))


def jet_fp8_linear_fwd(qx, sx, qw, sw, y, M, N, K, stream) -> int:
    return int(lib().jet_fp8_linear_fwd(qx, sx, qw, sw, y, M, N, K, stream))


def jet_fp8_linear_dgrad(qdy, sdy, qwT, swT, dx, M, N, K, stream) -> int:
    return int(lib().jet_fp8_linear_dgrad(qdy, sdy, qwT, swT, dx, M, N, K, stream))


def jet_fp8_linear_wgrad(qdyT, sdyT, qxT, sxT, dw, M, N, K, stream) -> int:
    return int(lib().jet_fp8_linear_wgrad(qdyT, sdyT, qxT, sxT, dw, M, N, K, stream))


def jet_rmsnorm_quant(x, gamma, eps, M, K, q_row, s_row, stream) -> int:
    return int(lib().jet_rmsnorm_quant(x, gamma, float(eps), M, K, q_row, s_row, stream))


def jet_silu_mul_quant(gate, up, ld, M, K, q_row, s_row, stream) -> int:
    return int(lib().jet_silu_mul_quant(gate, up, ld, M, K, q_row, s_row, stream))


def jet_silu_mul_bwd_quant(gate, up, ld, dh, M, K, dgu, q_row, s_row, q_colT, s_colT, stream) -> int:
    return int(lib().jet_silu_mul_bwd_quant(gate, up, ld, dh, M, K, dgu, q_row, s_row, q_colT, s_colT, stream))


def jet_silu_mul_bwd(gate, up, ld, dh, M, K, dgate, dup, ld_out, stream) -> int:
    return int(lib().jet_silu_mul_bwd(gate, up, ld, dh, M, K, dgate, dup, ld_out, stream))


# ------------------------------------------------------- tensor conveniences

def _stream() -> int:
    return torch.cuda.current_stream().cuda_stream


def _ptr(t):
    return None if t is None else t.data_ptr()


def _need(t: torch.Tensor, dtype, name: str):
    if not t.is_cuda or not t.is_contiguous() or t.dtype != dtype or t.dim() != 2:
        raise TypeError(f"{name}: need a contiguous 2-D CUDA tensor of {dtype}")


def _need_rows(t, dtype, rows: int, cols: int, like: torch.Tensor, name: str):
    """A quantizer's output (or the scales of its input) in the caller's tensor: the kernels go through
    [rows, cols] densely from data_ptr(), so it lies on the operand's device, is contiguous, has the element size and
    at least that many elements, and, unless it is flat, rows of `cols`.  More rows (a buffer of a larger batch) are fine.
    Codes may be in any one-byte type.  None is left to the C ABI."""
    if t is None:
        return
    fits = t.element_size() == 1 if dtype == torch.uint8 else t.dtype == dtype
    if not t.is_cuda or not t.is_contiguous() or not fits:
        raise TypeError(f"{name}: need a contiguous CUDA tensor of {dtype}")
    cols = max(cols, 1)
    if t.numel() < rows * cols or (t.dim() != 1 and (t.dim() == 0 or t.shape[-1] != cols)):
        raise ValueError(f"{name}: shape {tuple(t.shape)}, need {(rows, cols)}")
    if t.device != like.device:
        raise ValueError(f"{name}: on {t.device}, the operand on {like.device}")


def _need_row_pair(o: dict, M: int, K: int, like: torch.Tensor):
    _need_rows(o.get("q_row"), torch.uint8, M, K, like, "q_row")
    _need_rows(o.get("s_row"), torch.float32, M, K // GROUP, like, "s_row")


def _same_device(like: torch.Tensor, **others: torch.Tensor):
    for name, t in others.items():
        if t.device != like.device:
            raise ValueError(f"{name}: on {t.device}, the other operand on {like.device}")


def quant_act(x: torch.Tensor, x_scales: torch.Tensor | None = None, row: bool = True,
              col: bool = False, out: dict | None = None) -> dict:
    """1x128 quantization of a bf16 [M,K] tensor, or of an FP8-saved one (uint8 codes
    plus x_scales).  Returns dict(q_row, s_row, q_colT, s_colT) with the requested pairs."""
    r = (_host or _native()).quant_act(x, x_scales, row, col, out)
    if r is not None:
        return r
    src = JET_SRC_BF16 if x_scales is None else JET_SRC_FP8_ROW
    _need(x, torch.bfloat16 if src == JET_SRC_BF16 else torch.uint8, "x")
    M, K = x.shape
    dev = x.device
    if src == JET_SRC_FP8_ROW:
        _need_rows(x_scales, torch.float32, M, K // GROUP, x, "x_scales")
    o = {} if out is None else out
    if row and "q_row" not in o:
        o["q_row"] = torch.empty((M, K), dtype=torch.uint8, device=dev)
        o["s_row"] = torch.empty((M, max(K // GROUP, 1)), dtype=torch.float32, device=dev)
    if col and "q_colT" not in o:
        o["q_colT"] = torch.empty((K, M), dtype=torch.uint8, device=dev)
        o["s_colT"] = torch.empty((K, max(M // GROUP, 1)), dtype=torch.float32, device=dev)
    if row:
        _need_row_pair(o, M, K, x)
    if col:
        _need_rows(o.get("q_colT"), torch.uint8, K, M, x, "q_colT")
        _need_rows(o.get("s_colT"), torch.float32, K, M // GROUP, x, "s_colT")
    st = jet_quant_act(_ptr(x), _ptr(x_scales), src, M, K,
                       _ptr(o.get("q_row")) if row else None, _ptr(o.get("s_row")) if row else None,
                       _ptr(o.get("q_colT")) if col else None, _ptr(o.get("s_colT")) if col else None,
                       _stream())
    if st:
        raise JetError(st, "jet_quant_act")
    return o


def _row_pair(M, K, like, out):
    o = {} if out is None else out
    if "q_row" not in o:
        o["q_row"] = torch.empty((M, K), dtype=torch.uint8, device=like.device)
        o["s_row"] = torch.empty((M, max(K // GROUP, 1)), dtype=torch.float32, device=like.device)
    _need_row_pair(o, M, K, like)
    return o


def rmsnorm_quant(x: torch.Tensor, gamma: torch.Tensor, eps: float, out: dict | None = None) -> dict:
    """RMSNorm of bf16 [M,K] with bf16 weight [K], written as 1x128 FP8: dict(q_row, s_row)."""
    r = (_host or _native()).rmsnorm_quant(x, gamma, eps, out)
    if r is not None:
        return r
    _need(x, torch.bfloat16, "x")
    M, K = x.shape
    if not gamma.is_cuda or not gamma.is_contiguous() or gamma.dtype != torch.bfloat16 or gamma.shape != (K,):
        raise TypeError("gamma: need a contiguous CUDA bf16 tensor of K elements")
    _same_device(x, gamma=gamma)
    o = _row_pair(M, K, x, out)
    st = jet_rmsnorm_quant(_ptr(x), _ptr(gamma), eps, M, K, _ptr(o["q_row"]), _ptr(o["s_row"]), _stream())
    if st:
        raise JetError(st, "jet_rmsnorm_quant")
    return o


def silu_mul_quant(gate: torch.Tensor, up: torch.Tensor, out: dict | None = None) -> dict:
    """SiLU(gate) * up of two bf16 [M,K] tensors (contiguous, or the two halves of one
    contiguous [M,2K] tensor), written as 1x128 FP8: dict(q_row, s_row)."""
    r = (_host or _native()).silu_mul_quant(gate, up, out)
    if r is not None:
        return r
    for t, name in ((gate, "gate"), (up, "up")):
        if not t.is_cuda or t.dtype != torch.bfloat16 or t.dim() != 2 or t.stride(1) != 1:
            raise TypeError(f"{name}: need a 2-D CUDA bf16 tensor with unit column stride")
    if gate.shape != up.shape or gate.stride(0) != up.stride(0):
        raise TypeError("gate and up need one shape and one row stride")
    _same_device(gate, up=up)
    M, K = gate.shape
    o = _row_pair(M, K, gate, out)
    st = jet_silu_mul_quant(_ptr(gate), _ptr(up), gate.stride(0), M, K, _ptr(o["q_row"]), _ptr(o["s_row"]), _stream())
    if st:
        raise JetError(st, "jet_silu_mul_quant")
    return o


def silu_mul_bwd(gate: torch.Tensor, up: torch.Tensor, dh: torch.Tensor, out: torch.Tensor | None = None) -> torch.Tensor:
    """Backward of h = SiLU(gate) * up: returns dgu bf16 [M, 2K] = [dgate | dup] (one contiguous
    tensor, the layout the fused gate/up projection's backward consumes)."""
    r = (_host or _native()).silu_mul_bwd(gate, up, dh, out)
    if r is not None:
        return r
    for t, name in ((gate, "gate"), (up, "up")):
        if not t.is_cuda or t.dtype != torch.bfloat16 or t.dim() != 2 or t.stride(1) != 1:
            raise TypeError(f"{name}: need a 2-D CUDA bf16 tensor with unit column stride")
    if gate.shape != up.shape or gate.stride(0) != up.stride(0):
        raise TypeError("gate and up need one shape and one row stride")
    _need(dh, torch.bfloat16, "dh")
    M, K = gate.shape
    if tuple(dh.shape) != (M, K):
        raise ValueError("dh: need the shape of gate")
    dgu = torch.empty((M, 2 * K), dtype=torch.bfloat16, device=gate.device) if out is None else out
    _need(dgu, torch.bfloat16, "out")
    if tuple(dgu.shape) != (M, 2 * K):
        raise ValueError("out: need [M, 2K]")
    _same_device(gate, up=up, dh=dh, out=dgu)
    st = jet_silu_mul_bwd(_ptr(gate), _ptr(up), gate.stride(0), _ptr(dh), M, K, _ptr(dgu),
                          dgu.data_ptr() + 2 * K, 2 * K, _stream())
    if st:
        raise JetError(st, "jet_silu_mul_bwd")
    return dgu


def silu_mul_bwd_quant(gate: torch.Tensor, up: torch.Tensor, dh: torch.Tensor) -> tuple:
    """silu_mul_bwd and quant_act(dgu, row=True, col=True) in one pass: (dgu, dict(q_row, s_row, q_colT, s_colT))."""
    for t, name in ((gate, "gate"), (up, "up")):
        if not t.is_cuda or t.dtype != torch.bfloat16 or t.dim() != 2 or t.stride(1) != 1:
            raise TypeError(f"{name}: need a 2-D CUDA bf16 tensor with unit column stride")
    if gate.shape != up.shape or gate.stride(0) != up.stride(0):
        raise TypeError("gate and up need one shape and one row stride")
    _need(dh, torch.bfloat16, "dh")
    M, K = gate.shape
    if tuple(dh.shape) != (M, K):
        raise ValueError("dh: need the shape of gate")
    _same_device(gate, up=up, dh=dh)
    new = lambda rows, cols, dtype: torch.empty((rows, cols), dtype=dtype, device=gate.device)
    dgu = new(M, 2 * K, torch.bfloat16)
    o = dict(q_row=new(M, 2 * K, torch.uint8), s_row=new(M, max(2 * K // GROUP, 1), torch.float32),
             q_colT=new(2 * K, M, torch.uint8), s_colT=new(2 * K, max(M // GROUP, 1), torch.float32))
    st = jet_silu_mul_bwd_quant(_ptr(gate), _ptr(up), gate.stride(0), _ptr(dh), M, K, _ptr(dgu), _ptr(o["q_row"]),
                                _ptr(o["s_row"]), _ptr(o["q_colT"]), _ptr(o["s_colT"]), _stream())
    if st:
        raise JetError(st, "jet_silu_mul_bwd_quant")
    return dgu, o


def quant_weight(w: torch.Tensor, transposed: bool = False, out: tuple | None = None):
    """128x128 quantization of bf16 [N,K].  Returns (q, s) or (q, s, qT, sT)."""
    r = (_host or _native()).quant_weight(w, transposed, out)
    if r is not None:
        return r
    _need(w, torch.bfloat16, "w")
    N, K = w.shape
    dev = w.device
    if out is None:
        q = torch.empty((N, K), dtype=torch.uint8, device=dev)
        s = torch.empty((max(N // GROUP, 1), max(K // GROUP, 1)), dtype=torch.float32, device=dev)
        qT = torch.empty((K, N), dtype=torch.uint8, device=dev) if transposed else None
        sT = torch.empty((max(K // GROUP, 1), max(N // GROUP, 1)), dtype=torch.float32, device=dev) if transposed else None
    else:
        q, s, qT, sT = (tuple(out) + (None, None))[:4]
        _need_rows(q, torch.uint8, N, K, w, "q")
        _need_rows(s, torch.float32, N // GROUP, K // GROUP, w, "s")
        _need_rows(qT, torch.uint8, K, N, w, "qT")
        _need_rows(sT, torch.float32, K // GROUP, N // GROUP, w, "sT")
    st = jet_quant_weight(_ptr(w), N, K, _ptr(q), _ptr(s), _ptr(qT), _ptr(sT), _stream())
    if st:
        raise JetError(st, "jet_quant_weight")
    return (q, s, qT, sT) if transposed else (q, s)


def _need_operand(q, s, rows_per_scale: int, name: str):
    """FP8 codes [rows, R] with their scales [rows / rows_per_scale, R / 128]: the kernels read
    exactly these extents from the raw pointers, so a wrong dtype, a strided view or a scale
    array of another shape is refused here."""
    _need(q, torch.uint8, name)
    _need(s, torch.float32, name + " scales")
    rows, R = q.shape
    if R % GROUP or rows % rows_per_scale:
        raise ValueError(f"{name}: shape {tuple(q.shape)} does not divide into its scale groups")
    if tuple(s.shape) != (rows // rows_per_scale, R // GROUP):
        raise ValueError(f"{name} scales: shape {tuple(s.shape)}, need {(rows // rows_per_scale, R // GROUP)}")
    if s.device != q.device:
        raise ValueError(f"{name}: codes and scales on different devices")


def _gemm_out(out, shape, a, b, name: str) -> torch.Tensor:
    if a.shape[1] != b.shape[1]:
        raise ValueError(f"{name}: reduction lengths differ ({a.shape[1]} and {b.shape[1]})")
    if a.device != b.device:
        raise ValueError(f"{name}: operands on different devices")
    if out is None:
        return torch.empty(shape, dtype=torch.bfloat16, device=a.device)
    _need(out, torch.bfloat16, name + " out")
    if tuple(out.shape) != tuple(shape) or out.device != a.device:
        raise ValueError(f"{name} out: shape {tuple(out.shape)} on {out.device}, need {tuple(shape)} on {a.device}")
    return out


def fp8_linear_fwd(qx, sx, qw, sw, out: torch.Tensor | None = None) -> torch.Tensor:
    """y bf16 [M,N] = X W^T."""
    r = (_host or _native()).gemm(0, qx, sx, qw, sw, out)
    if r is not None:
        return r
    _need_operand(qx, sx, 1, "qx")
    _need_operand(qw, sw, GROUP, "qw")
    M, K = qx.shape
    N = qw.shape[0]
    y = _gemm_out(out, (M, N), qx, qw, "fp8_linear_fwd")
    st = jet_fp8_linear_fwd(_ptr(qx), _ptr(sx), _ptr(qw), _ptr(sw), _ptr(y), M, N, K, _stream())
    if st:
        raise JetError(st, "jet_fp8_linear_fwd")
    return y


def fp8_linear_dgrad(qdy, sdy, qwT, swT, out: torch.Tensor | None = None) -> torch.Tensor:
    """dx bf16 [M,K] = dY W."""
    r = (_host or _native()).gemm(1, qdy, sdy, qwT, swT, out)
    if r is not None:
        return r
    _need_operand(qdy, sdy, 1, "qdy")
    _need_operand(qwT, swT, GROUP, "qwT")
    M, N = qdy.shape
    K = qwT.shape[0]
    dx = _gemm_out(out, (M, K), qdy, qwT, "fp8_linear_dgrad")
    st = jet_fp8_linear_dgrad(_ptr(qdy), _ptr(sdy), _ptr(qwT), _ptr(swT), _ptr(dx), M, N, K, _stream())
    if st:
        raise JetError(st, "jet_fp8_linear_dgrad")
    return dx


def fp8_linear_wgrad(qdyT, sdyT, qxT, sxT, out: torch.Tensor | None = None) -> torch.Tensor:
    """dw bf16 [N,K] = dY^T X."""
    r = (_host or _native()).gemm(2, qdyT, sdyT, qxT, sxT, out)
    if r is not None:
        return r
    _need_operand(qdyT, sdyT, 1, "qdyT")
    _need_operand(qxT, sxT, 1, "qxT")
    N, M = qdyT.shape
    K = qxT.shape[0]
    dw = _gemm_out(out, (N, K), qdyT, qxT, "fp8_linear_wgrad")
    st = jet_fp8_linear_wgrad(_ptr(qdyT), _ptr(sdyT), _ptr(qxT), _ptr(sxT), _ptr(dw), M, N, K, _stream())
    if st:
        raise JetError(st, "jet_fp8_linear_wgrad")
    return dw
