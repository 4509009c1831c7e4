"""Thin binding of the C-ABI library libfcv2 (include/fcv2.h).  Same names as the C entry points.

Argument marshalling only: torch supplies device memory and the current HIP stream, every step of the codec
runs in the library's kernels.  The calls that launch kernels are marshalled by the native module _fcv2_torch
(csrc/fcv2_torch.cpp: a decode-sized call spends less time on the GPU than Python needs to read its tensors); the host-only
ones go through ctypes.  There is no CPU fallback: if the library or its binding cannot be loaded, calls raise.
"""
import ctypes as C
import importlib.util
import os
from dataclasses import dataclass

import torch

from . import build as _build

F_SPIKE = 1
F_META_FP32 = 2
F_META_INT = 4
F_IDX_BF16 = 8
DT_BF16 = 0
DT_FP32 = 1
ABSENT = 2**64 - 1
TENSOR_ALIGN = 256
ROW_ALIGN = 16
MAX_PEERS = 16
STATIC_SCRATCH_BYTES = 2 << 20


class Fcv2Error(RuntimeError):
    pass


class _Fmt(C.Structure):
    _fields_ = [("bits", C.c_uint32), ("group", C.c_uint32), ("flags", C.c_uint32)]


class _Layout(C.Structure):
    _fields_ = [(k, C.c_uint64) for k in (
        "n", "n_groups", "total_bytes", "off_plane8", "off_plane4", "off_plane2", "off_plane1",
        "off_scale", "off_zero", "off_spike_val", "off_spike_idx")]


@dataclass(frozen=True)
class Layout:
    n: int
    n_groups: int
    total_bytes: int
    off_plane8: int
    off_plane4: int
    off_plane2: int
    off_plane1: int
    off_scale: int
    off_zero: int
    off_spike_val: int
    off_spike_idx: int


_lib = None
_native = None  # the module _fcv2_torch once it is loaded


def lib():
    """Load libfcv2.so.  A built library that matches the sources is loaded as it is; a missing one, or one built from
    other sources than the tree now holds (an edit since the last build), is compiled first.  A failing compile raises:
    there is no other path."""
    global _lib
    if _lib is None:
        path = _build.lib_path()
        if not os.path.exists(path) or not _build.is_current():
            _build.build()
        L = C.CDLL(path)
        fmtp, vp = C.POINTER(_Fmt), C.c_void_p
        L.fcv2_get_layout.argtypes = [C.c_uint64, fmtp, C.c_uint32, C.POINTER(_Layout)]
        L.fcv2_quantize_pack.argtypes = [vp, C.c_uint64, fmtp, vp, vp]
        L.fcv2_unpack_dequant.argtypes = [vp, C.c_uint64, fmtp, vp, C.c_int, vp]
        L.fcv2_quantize_pack_slices.argtypes = [vp, C.c_uint64, C.c_uint32, fmtp, vp, C.c_uint64, vp]
        L.fcv2_unpack_dequant_slices.argtypes = [C.POINTER(vp), C.c_uint32, C.c_uint64, fmtp, vp, C.c_int, vp]
        L.fcv2_stream_copy.argtypes = [vp, vp, C.c_uint64, vp]  # include/fcv2_diag.h
        L.fcv2_reduce_requant.argtypes = [C.POINTER(vp), C.c_int, C.c_uint64, fmtp, fmtp, vp, vp, vp]
        L.fcv2_dispatch_workspace_bytes.argtypes = [C.c_uint32, C.c_uint32, C.c_uint32, C.POINTER(C.c_size_t)]
        L.fcv2_dispatch_quant.argtypes = [vp, vp, C.c_uint32, C.c_uint32, C.c_uint32, C.c_uint32, fmtp, vp, vp, vp,
                                          vp, C.c_size_t, vp]
        L.fcv2_dispatch_quant_noalloc.argtypes = [vp, vp, C.c_uint32, C.c_uint32, C.c_uint32, C.c_uint32, fmtp, vp, vp, vp, vp]
        L.fcv2_status_string.argtypes = [C.c_int]
        L.fcv2_status_string.restype = C.c_char_p
        L.fcv2_version.restype = C.c_int
        _lib = L
    return _lib


def _check(rc, what):
    if rc != 0:
        raise Fcv2Error(f"{what}: {lib().fcv2_status_string(rc).decode()} ({rc})")


def _load_native():
    """The native binding, loaded on first use (after libfcv2.so, which lib() compiles together with it if need be)."""
    global _native
    if _native is None:
        lib()
        spec = importlib.util.spec_from_file_location("_fcv2_torch", _build.BINDING)
        m = importlib.util.module_from_spec(spec)
        spec.loader.exec_module(m)
        m.set_errors(Fcv2Error, torch.OutOfMemoryError)
        _native = m
    return _native


def _stream():
    return C.c_void_p(torch.cuda.current_stream().cuda_stream)


def _dev(t: torch.Tensor, what: str):
    if not t.is_cuda or not t.is_contiguous():
        raise Fcv2Error(f"{what} must be a contiguous device tensor")
    return C.c_void_p(t.data_ptr())


def version() -> int:
    return lib().fcv2_version()


def get_layout(n, bits, group, flags, section_align=TENSOR_ALIGN) -> Layout:
    out = _Layout()
    _check(lib().fcv2_get_layout(n, C.byref(_Fmt(bits, group, flags)), section_align, C.byref(out)), "fcv2_get_layout")
    return Layout(*(getattr(out, k) for k, _ in _Layout._fields_))


def quantize_pack(x: torch.Tensor, bits, group, flags, out: torch.Tensor = None) -> torch.Tensor:
    """x: bf16 device tensor (any shape, contiguous).  Returns the packed record as a uint8 device tensor."""
    return (_native or _load_native()).quantize_pack(x, bits, group, flags, out)


def unpack_dequant(packed: torch.Tensor, n, bits, group, flags, out_dtype=torch.float32,
                   out: torch.Tensor = None) -> torch.Tensor:
    return (_native or _load_native()).unpack_dequant(packed, n, bits, group, flags, out_dtype, out)


def quantize_pack_slices(x: torch.Tensor, n_slices, bits, group, flags, out: torch.Tensor = None) -> torch.Tensor:
    """Cut x into n_slices equal slices and pack each into a record of its own.  Returns a uint8 tensor
    [n_slices, record_stride]; row j is the record of slice j."""
    return (_native or _load_native()).quantize_pack_slices(x, n_slices, bits, group, flags, out)


def unpack_dequant_slices(records, n, bits, group, flags, out_dtype=torch.float32, out: torch.Tensor = None) -> torch.Tensor:
    """records: list of packed uint8 device tensors, record j = slice j of the output of n elements."""
    return (_native or _load_native()).unpack_dequant_slices(records, n, bits, group, flags, out_dtype, out)


def stream_copy(src: torch.Tensor, dst: torch.Tensor):
    """Diagnostic: plain streaming copy of src into dst (same byte size, a multiple of 16)."""
    nbytes = src.numel() * src.element_size()
    if nbytes != dst.numel() * dst.element_size():
        raise Fcv2Error("src and dst differ in size")
    _check(lib().fcv2_stream_copy(_dev(src, "src"), _dev(dst, "dst"), nbytes, _stream()), "fcv2_stream_copy")


def reduce_requant(peers, n, fmt_in, fmt_out=None, want_sum=False, out: torch.Tensor = None,
                   sum_out: torch.Tensor = None):
    """peers: list of packed uint8 device tensors of format fmt_in = (bits, group, flags).
    Returns packed_out, or (packed_out, fp32 sums) with want_sum."""
    return (_native or _load_native()).reduce_requant(peers, n, fmt_in, fmt_out, want_sum, out, sum_out)


def dispatch_workspace_bytes(T, K, E) -> int:
    out = C.c_size_t()
    _check(lib().fcv2_dispatch_workspace_bytes(T, K, E, C.byref(out)), "fcv2_dispatch_workspace_bytes")
    return out.value


def dispatch_quant(x: torch.Tensor, topk_ids: torch.Tensor, E, bits, group, flags, send_buf=None,
                   expert_offsets=None, row_src=None, workspace=None):
    """x: [T, H] bf16, topk_ids: [T, K] int32 (device).  Returns send_buf [T*K, row_bytes] uint8,
    expert_offsets [E+1] int32, row_src [T*K] int32 (first expert_offsets[E] entries valid)."""
    return (_native or _load_native()).dispatch_quant(x, topk_ids, E, bits, group, flags, send_buf, expert_offsets, row_src, workspace)


def dispatch_quant_noalloc(x: torch.Tensor, topk_ids: torch.Tensor, E, bits, group, flags, send_buf: torch.Tensor,
                           expert_offsets: torch.Tensor, row_src: torch.Tensor):
    """fcv2_dispatch_quant_noalloc: as dispatch_quant, but the planning scratch is the library's static device array.
    The caller passes every output; this binding allocates nothing either."""
    return (_native or _load_native()).dispatch_quant_noalloc(x, topk_ids, E, bits, group, flags, send_buf, expert_offsets, row_src)
