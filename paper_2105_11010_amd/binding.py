"""Binding of libsparq.so -- argument marshalling only: ctypes here, and _sparq_native.so (csrc/binding/sparq_native.cpp) for the
calls a program makes per layer.

Function names and arguments mirror include/sparq.h.  Tensors are torch CUDA
(ROCm) tensors used purely as device buffers; every step of the computation
runs inside the library's HIP kernels.  There is no CPU fallback: if the
library has not been built, importing this module raises.
"""
from __future__ import annotations

import ctypes
import os
from typing import Optional

import torch

_HERE = os.path.dirname(os.path.abspath(__file__))
# SPARQ_LIBRARY points at another build of the same library (A/B comparisons); default: the in-tree build
LIB_PATH = os.environ.get("SPARQ_LIBRARY") or os.path.join(_HERE, "libsparq.so")

SPARQ_OK, SPARQ_EINVAL, SPARQ_EUNSUPPORTED, SPARQ_EWORKSPACE, SPARQ_ELAUNCH = range(5)


class SparqMode(ctypes.Structure):
    _fields_ = [("window_bits", ctypes.c_int32), ("shift_mask", ctypes.c_uint32),
                ("round_nearest", ctypes.c_int32), ("pair", ctypes.c_int32)]


class SparqConvDesc(ctypes.Structure):
    _fields_ = [(k, ctypes.c_int32) for k in
                ("B", "H", "W", "C", "N", "KH", "KW", "stride_h", "stride_w", "pad_h", "pad_w")]


class SparqError(RuntimeError):
    def __init__(self, status: int, what: str):
        self.status = status
        super().__init__(f"{what}: {strerror(status)} (status {status})")


def _load() -> ctypes.CDLL:
    if not os.path.exists(LIB_PATH):
        raise ImportError(f"{LIB_PATH} not built; run `python -c 'import __graft_entry__ as g; g.build()'`")
    L = ctypes.CDLL(LIB_PATH)
    vp, i64, i32, sz = ctypes.c_void_p, ctypes.c_int64, ctypes.c_int32, ctypes.c_size_t
    pm, pd = ctypes.POINTER(SparqMode), ctypes.POINTER(SparqConvDesc)
    L.sparq_trim.argtypes = [vp, vp, i64, i32, pm, vp]
    L.sparq_trim.restype = ctypes.c_int
    L.sparq_packed_bytes.argtypes = [pd]
    L.sparq_packed_bytes.restype = sz
    L.sparq_pack_weights.argtypes = [vp, pd, vp, sz, vp]
    L.sparq_pack_weights.restype = ctypes.c_int
    L.sparq_workspace_bytes.argtypes = [pd, pm]
    L.sparq_workspace_bytes.restype = sz
    L.sparq_conv_plan.argtypes = [pd, pm, ctypes.c_char_p, sz]
    L.sparq_conv_plan.restype = ctypes.c_int
    L.sparq_sparse24_plan.argtypes = [pd, pm, ctypes.c_char_p, sz]
    L.sparq_sparse24_plan.restype = ctypes.c_int
    L.sparq_conv_gemm.argtypes = [vp, vp, pd, pm, vp, vp, vp, vp, sz, vp]
    L.sparq_conv_gemm.restype = ctypes.c_int
    L.sparq_conv_gemm_static_ws.argtypes = [vp, vp, pd, pm, vp, vp, vp, vp]
    L.sparq_conv_gemm_static_ws.restype = ctypes.c_int
    L.sparq_dequant.argtypes = [vp, vp, vp, i64, i32, vp]
    L.sparq_dequant.restype = ctypes.c_int
    L.sparq_conv_gemm_u8.argtypes = [vp, vp, pd, pm, vp, vp, pm, vp, sz, vp]
    L.sparq_conv_gemm_u8.restype = ctypes.c_int
    L.sparq_requant.argtypes = [vp, vp, vp, i64, i32, vp]
    L.sparq_requant.restype = ctypes.c_int
    L.sparq_packed_act_bytes.argtypes = [i64, i32, pm, i32]
    L.sparq_packed_act_bytes.restype = sz
    L.sparq_pack_act.argtypes = [vp, vp, sz, i64, i32, pm, i32, vp]
    L.sparq_pack_act.restype = ctypes.c_int
    L.sparq_unpack_act.argtypes = [vp, sz, vp, i64, i32, pm, i32, vp]
    L.sparq_unpack_act.restype = ctypes.c_int
    L.sparq_conv_packed_workspace_bytes.argtypes = [pd, pm]
    L.sparq_conv_packed_workspace_bytes.restype = sz
    L.sparq_conv_gemm_packed.argtypes = [vp, sz, i32, vp, pd, pm, vp, vp, vp, vp, sz, vp]
    L.sparq_conv_gemm_packed.restype = ctypes.c_int
    L.sparq_sparse24_packed_bytes.argtypes = [pd, pm]
    L.sparq_sparse24_packed_bytes.restype = sz
    L.sparq_pack_weights_sparse24.argtypes = [vp, vp, pd, pm, vp, sz, vp]
    L.sparq_pack_weights_sparse24.restype = ctypes.c_int
    L.sparq_sparse24_workspace_bytes.argtypes = [pd, pm]
    L.sparq_sparse24_workspace_bytes.restype = sz
    L.sparq_conv_gemm_sparse24.argtypes = [vp, vp, pd, pm, vp, vp, vp, vp, sz, vp]
    L.sparq_conv_gemm_sparse24.restype = ctypes.c_int
    L.sparq_set_tuning.argtypes = [ctypes.c_char_p]
    L.sparq_set_tuning.restype = ctypes.c_int
    L.sparq_strerror.argtypes = [ctypes.c_int]
    L.sparq_strerror.restype = ctypes.c_char_p
    return L


lib = _load()


def _load_native():
    """The per-layer entry points, on the library loaded above."""
    try:
        from . import _sparq_native as n
    except ImportError as e:
        raise ImportError(f"_sparq_native.so not built; run `python -c 'import __graft_entry__ as g; g.build()'` ({e})") from e
    names = ("trim", "conv_gemm", "conv_gemm_u8", "conv_gemm_packed", "conv_gemm_sparse24", "dequant", "requant", "pack_act", "unpack_act")
    n.bind(tuple(ctypes.cast(getattr(lib, "sparq_" + k), ctypes.c_void_p).value for k in names), SparqMode, SparqConvDesc, SparqError)
    return n


_native = _load_native()
sparq_trim = _native.sparq_trim
sparq_conv_gemm = _native.sparq_conv_gemm
sparq_conv_gemm_u8 = _native.sparq_conv_gemm_u8
sparq_conv_gemm_packed = _native.sparq_conv_gemm_packed
sparq_conv_gemm_sparse24 = _native.sparq_conv_gemm_sparse24
sparq_dequant = _native.sparq_dequant
sparq_requant = _native.sparq_requant
sparq_pack_act = _native.sparq_pack_act
sparq_unpack_act = _native.sparq_unpack_act


def strerror(status: int) -> str:
    return lib.sparq_strerror(int(status)).decode()


def mode(window_bits: int = 4, shift_mask: int = 0x1F, round_nearest: int = 0, pair: int = 1) -> SparqMode:
    return SparqMode(int(window_bits), int(shift_mask), int(round_nearest), int(pair))


def conv_desc(B, H, W, C, N, KH=1, KW=1, stride=(1, 1), pad=(0, 0)) -> SparqConvDesc:
    return SparqConvDesc(B, H, W, C, N, KH, KW, stride[0], stride[1], pad[0], pad[1])


def out_rows(d: SparqConvDesc) -> int:
    Ho = (d.H + 2 * d.pad_h - d.KH) // d.stride_h + 1
    Wo = (d.W + 2 * d.pad_w - d.KW) // d.stride_w + 1
    return d.B * Ho * Wo


# Address of a device's current stream, without the Stream object torch.cuda.current_stream() builds for it (2.9 us of a
# 9 us call; 0.1 this way).
_current_raw_stream = torch._C._cuda_getCurrentRawStream if hasattr(torch._C, "_cuda_getCurrentRawStream") else None


def _stream() -> int:
    if _current_raw_stream is None:
        return torch.cuda.current_stream().cuda_stream
    return _current_raw_stream(torch.cuda.current_device())


def _dev(t: Optional[torch.Tensor], dtype, name: str) -> Optional[int]:
    if t is None:
        return None
    if not t.is_cuda or t.dtype != dtype or not t.is_contiguous():
        raise TypeError(f"{name} must be a contiguous device tensor of dtype {dtype}")
    return t.data_ptr()


def _check(status: int, what: str) -> None:
    if status != SPARQ_OK:
        raise SparqError(status, what)


def sparq_packed_bytes(d: SparqConvDesc) -> int:
    return int(lib.sparq_packed_bytes(ctypes.byref(d)))


def sparq_workspace_bytes(d: SparqConvDesc, m: SparqMode) -> int:
    return int(lib.sparq_workspace_bytes(ctypes.byref(d), ctypes.byref(m)))


def sparq_conv_plan(d: SparqConvDesc, m: SparqMode) -> str:
    """Which kernel and tiling sparq_conv_gemm would use (a line of text for logs)."""
    buf = ctypes.create_string_buffer(256)
    _check(lib.sparq_conv_plan(ctypes.byref(d), ctypes.byref(m), buf, len(buf)), "sparq_conv_plan")
    return buf.value.decode()


def sparq_sparse24_plan(d: SparqConvDesc, m: SparqMode) -> str:
    """Which kernel sparq_conv_gemm_sparse24 would use, and on which matrix instruction (a line of text for logs)."""
    buf = ctypes.create_string_buffer(256)
    _check(lib.sparq_sparse24_plan(ctypes.byref(d), ctypes.byref(m), buf, len(buf)), "sparq_sparse24_plan")
    return buf.value.decode()


def sparq_pack_weights(w: torch.Tensor, d: SparqConvDesc, packed: torch.Tensor) -> None:
    """w int8 [N,KH,KW,C] -> packed (uint8 device buffer of sparq_packed_bytes(d))."""
    if tuple(w.shape) != (d.N, d.KH, d.KW, d.C):
        raise ValueError("weight shape does not match the descriptor")
    _check(lib.sparq_pack_weights(_dev(w, torch.int8, "w"), ctypes.byref(d), _dev(packed, torch.uint8, "packed"),
                                  packed.numel(), _stream()), "sparq_pack_weights")


def sparq_conv_gemm_static_ws(x: torch.Tensor, packed: torch.Tensor, d: SparqConvDesc, m: SparqMode,
                              acc: Optional[torch.Tensor] = None, scale: Optional[torch.Tensor] = None,
                              out: Optional[torch.Tensor] = None) -> None:
    """sparq_conv_gemm with its scratch taken from the library's own per-GPU array (nothing is allocated)."""
    if x.numel() != d.B * d.H * d.W * d.C:
        raise ValueError("activation size does not match the descriptor")
    M = out_rows(d)
    for t, nm in ((acc, "acc"), (out, "out")):
        if t is not None and t.numel() != M * d.N:
            raise ValueError(f"{nm} must hold M*N = {M * d.N} elements")
    if scale is not None and scale.numel() != d.N:
        raise ValueError("scale must hold N elements")
    _check(lib.sparq_conv_gemm_static_ws(_dev(x, torch.uint8, "x"), _dev(packed, torch.uint8, "packed"), ctypes.byref(d),
                                         ctypes.byref(m), _dev(acc, torch.int32, "acc"),
                                         _dev(scale, torch.float32, "scale"), _dev(out, torch.float32, "out"), _stream()),
           "sparq_conv_gemm_static_ws")


def sparq_packed_act_bytes(rows: int, C: int, m: SparqMode, group: int = 1) -> int:
    """Bytes of the packed form of [rows][C] activations (0: this mode / group has none)."""
    return int(lib.sparq_packed_act_bytes(int(rows), int(C), ctypes.byref(m), int(group)))


def sparq_conv_packed_workspace_bytes(d: SparqConvDesc, m: SparqMode) -> int:
    return int(lib.sparq_conv_packed_workspace_bytes(ctypes.byref(d), ctypes.byref(m)))


def sparq_sparse24_packed_bytes(d: SparqConvDesc, m: SparqMode) -> int:
    return int(lib.sparq_sparse24_packed_bytes(ctypes.byref(d), ctypes.byref(m)))


def sparq_sparse24_workspace_bytes(d: SparqConvDesc, m: SparqMode) -> int:
    return int(lib.sparq_sparse24_workspace_bytes(ctypes.byref(d), ctypes.byref(m)))


def sparq_pack_weights_sparse24(w_vals: torch.Tensor, w_idx: torch.Tensor, d: SparqConvDesc, m: SparqMode,
                                packed: torch.Tensor) -> None:
    """2:4 compressed weights (values int8 and coordinates uint8, both [N,KH,KW,C/2]) -> packed device buffer."""
    if tuple(w_vals.shape) != (d.N, d.KH, d.KW, d.C // 2) or w_idx.shape != w_vals.shape:
        raise ValueError("weight shapes do not match the descriptor")
    _check(lib.sparq_pack_weights_sparse24(_dev(w_vals, torch.int8, "w_vals"), _dev(w_idx, torch.uint8, "w_idx"),
                                           ctypes.byref(d), ctypes.byref(m), _dev(packed, torch.uint8, "packed"),
                                           packed.numel(), _stream()), "sparq_pack_weights_sparse24")


def sparq_set_tuning(spec: Optional[str] = None) -> None:
    """Test / tuning hook: force the kernel choice ("path=patch,patch_tn=128,patch_ws=1", "form=rows", ...); None clears it."""
    _check(lib.sparq_set_tuning(spec.encode() if spec else None), "sparq_set_tuning")
