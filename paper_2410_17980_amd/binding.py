"""Thin binding of libsbattn.so (include/sb_attn.h, include/sb_diag.h): same names, argument
marshalling only.  torch is used to own device memory and to name the stream;
every step of the computation runs inside the library's kernels.

The calls of the method are marshalled by a small native module (csrc/sb_torch.cpp), the
measurement aids and load()'s handle by ctypes.  Enqueue time of one call, ctypes -> native:
decode 16.9 -> 6.8 us, a short forward 11.5 -> 4.3 us, forward and backward 46 -> 18 us (kernels
launched by them: 2, 1, 5); the kernels of such calls run for 5 to 10 us, so the host set the pace.

There is no fallback: if the library is missing or a call fails, this raises.
"""
from __future__ import annotations

import ctypes
import importlib.util
import os

import torch

_HERE = os.path.dirname(os.path.abspath(__file__))
LIB_PATH = os.path.join(_HERE, "libsbattn.so")
EXT_PATH = os.path.join(_HERE, "_sbtorch.so")

EXPORTS = (
    "sb_attn_fwd", "sb_attn_fwd_halt", "sb_attn_fwd_train", "sb_attn_fwd_f32",
    "sb_attn_bwd_workspace_bytes", "sb_attn_bwd_gqa_workspace_bytes", "sb_attn_bwd", "sb_attn_bwd_dq", "sb_attn_bwd_dkdv",
    "sb_attn_fwd_rb", "sb_attn_bwd_rb", "sb_attn_fwd_gqa", "sb_attn_bwd_gqa",
    "sb_attn_varlen_fwd", "sb_attn_varlen_bwd_workspace_bytes", "sb_attn_varlen_bwd_gqa_workspace_bytes", "sb_attn_varlen_bwd",
    "sb_attn_decode_workspace_bytes", "sb_attn_decode", "sb_attn_decode_static",
    "sb_diag_mfma_rate", "sb_diag_stream_read", "sb_diag_fwd_clock", "sb_diag_fwd_tri",
    "sb_status_string", "sb_version",
)

_lib = None
_ext = None


class SbAttnError(RuntimeError):
    pass


def load(build_if_missing: bool = True):
    """Load libsbattn.so (building it first only when no built library exists)."""
    global _lib
    if _lib is not None:
        return _lib
    missing = [p for p in (LIB_PATH, EXT_PATH) if not os.path.exists(p)]
    if missing:
        if not build_if_missing:
            raise SbAttnError(f"{missing[0]} not built; run `python -m paper_2410_17980_amd.build`")
        from . import build as _build
        _build.build()
    lib = ctypes.CDLL(LIB_PATH)
    vp, ci, fp = ctypes.c_void_p, ctypes.c_int, ctypes.c_void_p
    lib.sb_attn_fwd.argtypes = [vp, vp, vp, vp, ci, ci, ci, ci, vp]
    lib.sb_attn_fwd.restype = ci
    lib.sb_attn_fwd_halt.argtypes = [vp, vp, vp, vp, ctypes.c_float, vp, ci, ci, ci, ci, vp]
    lib.sb_attn_fwd_halt.restype = ci
    lib.sb_attn_fwd_train.argtypes = [vp, vp, vp, vp, fp, ci, ci, ci, ci, vp]
    lib.sb_attn_fwd_train.restype = ci
    lib.sb_attn_fwd_f32.argtypes = [fp, fp, fp, fp, fp, ci, ci, ci, ci, vp]
    lib.sb_attn_fwd_f32.restype = ci
    lib.sb_attn_bwd_workspace_bytes.argtypes = [ci, ci, ci, ci]
    lib.sb_attn_bwd_workspace_bytes.restype = ctypes.c_size_t
    lib.sb_attn_bwd_gqa_workspace_bytes.argtypes = [ci, ci, ci, ci, ci]
    lib.sb_attn_bwd_gqa_workspace_bytes.restype = ctypes.c_size_t
    lib.sb_attn_bwd.argtypes = [vp, vp, vp, fp, vp, fp, fp, fp, vp, ctypes.c_size_t, ci, ci, ci, ci, vp]
    lib.sb_attn_bwd.restype = ci
    lib.sb_attn_bwd_dq.argtypes = [vp, vp, vp, fp, vp, fp, vp, ctypes.c_size_t, ci, ci, ci, ci, vp]
    lib.sb_attn_bwd_dq.restype = ci
    lib.sb_attn_bwd_dkdv.argtypes = [vp, vp, vp, vp, fp, fp, vp, ctypes.c_size_t, ci, ci, ci, ci, vp]
    lib.sb_attn_bwd_dkdv.restype = ci
    lib.sb_attn_fwd_rb.argtypes = [vp, vp, vp, vp, vp, fp, ci, ci, ci, ci, vp]
    lib.sb_attn_fwd_rb.restype = ci
    lib.sb_attn_bwd_rb.argtypes = [vp, vp, vp, vp, fp, vp, fp, fp, fp, fp, vp, ctypes.c_size_t, ci, ci, ci, ci, vp]
    lib.sb_attn_bwd_rb.restype = ci
    lib.sb_attn_fwd_gqa.argtypes = [vp, vp, vp, vp, vp, fp, ci, ci, ci, ci, ci, vp]
    lib.sb_attn_fwd_gqa.restype = ci
    lib.sb_attn_bwd_gqa.argtypes = [vp, vp, vp, vp, fp, vp, fp, fp, fp, fp, vp, ctypes.c_size_t,
                                    ci, ci, ci, ci, ci, vp]
    lib.sb_attn_bwd_gqa.restype = ci
    lib.sb_attn_varlen_fwd.argtypes = [vp, vp, vp, vp, vp, fp, vp, ci, ci, ci, ci, ci, ci, vp]
    lib.sb_attn_varlen_fwd.restype = ci
    lib.sb_attn_varlen_bwd_workspace_bytes.argtypes = [ci, ci, ci, ci, ci]
    lib.sb_attn_varlen_bwd_workspace_bytes.restype = ctypes.c_size_t
    lib.sb_attn_varlen_bwd_gqa_workspace_bytes.argtypes = [ci, ci, ci, ci, ci, ci]
    lib.sb_attn_varlen_bwd_gqa_workspace_bytes.restype = ctypes.c_size_t
    lib.sb_attn_varlen_bwd.argtypes = [vp, vp, vp, vp, fp, vp, fp, fp, fp, fp, vp, ci, ci, ci, ci, ci, ci,
                                       vp, ctypes.c_size_t, vp]
    lib.sb_attn_varlen_bwd.restype = ci
    lib.sb_attn_decode_workspace_bytes.argtypes = [ci, ci, ci, ci]
    lib.sb_attn_decode_workspace_bytes.restype = ctypes.c_size_t
    lib.sb_attn_decode.argtypes = [vp, vp, vp, vp, vp, fp, vp, ctypes.c_size_t, ci, ci, ci, ci, ci, ci, vp]
    lib.sb_attn_decode.restype = ci
    lib.sb_attn_decode_static.argtypes = [vp, vp, vp, vp, vp, fp, ci, ci, ci, ci, ci, ci, vp]
    lib.sb_attn_decode_static.restype = ci
    lib.sb_diag_mfma_rate.argtypes = [vp, ctypes.c_size_t, ci, vp, ctypes.POINTER(ctypes.c_double), vp]
    lib.sb_diag_mfma_rate.restype = ci
    lib.sb_diag_stream_read.argtypes = [vp, ctypes.c_size_t, vp, vp]
    lib.sb_diag_stream_read.restype = ci
    lib.sb_diag_fwd_clock.argtypes = [vp, vp, vp, vp, fp, ci, ci, ci, ci, vp, vp]
    lib.sb_diag_fwd_clock.restype = ci
    lib.sb_diag_fwd_tri.argtypes = [vp, vp, vp, vp, fp, ci, ci, ci, ci, vp]
    lib.sb_diag_fwd_tri.restype = ci
    lib.sb_status_string.argtypes = [ci]
    lib.sb_status_string.restype = ctypes.c_char_p
    lib.sb_version.argtypes = []
    lib.sb_version.restype = ci
    _lib = lib
    return lib


def _load_ext():
    global _ext
    load()
    spec = importlib.util.spec_from_file_location("_sbtorch", EXT_PATH)
    ext = importlib.util.module_from_spec(spec)
    spec.loader.exec_module(ext)
    ext.set_errors(SbAttnError, torch.cuda.OutOfMemoryError)
    _ext = ext
    return ext


def sb_status_string(status: int) -> str:
    return load().sb_status_string(int(status)).decode()


def sb_version() -> int:
    return int(load().sb_version())


def _check(rc: int, what: str):
    if rc != 0:
        raise SbAttnError(f"{what} failed: {sb_status_string(rc)} ({rc})")


def _dims(t: torch.Tensor):
    if t.dim() != 4:
        raise SbAttnError("expected a [B, H, T, d] tensor")
    return tuple(int(x) for x in t.shape)


def _ptr(t, dtype, shape=None, name="tensor"):
    if t is None:
        return None
    if not t.is_cuda:
        raise SbAttnError(f"{name} must live on the GPU")
    if t.dtype != dtype:
        raise SbAttnError(f"{name} must be {dtype}, got {t.dtype}")
    if not t.is_contiguous():
        raise SbAttnError(f"{name} must be contiguous")
    if shape is not None and tuple(t.shape) != tuple(shape):
        raise SbAttnError(f"{name} has shape {tuple(t.shape)}, expected {tuple(shape)}")
    return ctypes.c_void_p(t.data_ptr())


def _on(stream):
    """`stream` as the current one, for what a measurement allocates, fills and reads back."""
    if stream is not None and not isinstance(stream, torch.cuda.Stream):
        stream = torch.cuda.ExternalStream(stream.cuda_stream)
    return torch.cuda.stream(stream)


def _stream():
    return ctypes.c_void_p(torch.cuda.current_stream().cuda_stream)


# The calls of the method go through the native module: it checks the tensors, allocates what was
# not passed in, takes the stream and calls the C ABI (csrc/sb_torch.cpp).  With stream= a call launches and
# allocates as under `with torch.cuda.stream(stream)`, and what it returns may be dropped while work of the stream that was
# current still uses it.


def sb_attn_fwd(q, k, v, o=None, stream=None):
    """bf16 forward.  Returns o (allocated when not given)."""
    return (_ext or _load_ext()).forward("sb_attn_fwd", False, q, k, v, None, o, None, False, stream)


def sb_attn_fwd_halt(q, k, v, eps, o=None, tile_counts=None, stream=None):
    """bf16 forward with early halt.  tile_counts: optional int64 tensor of 2 on the GPU (added to)."""
    return (_ext or _load_ext()).halt(q, k, v, eps, o, tile_counts, stream)


def sb_attn_fwd_train(q, k, v, o=None, m=None, stream=None):
    """bf16 forward that also returns m[B,H,T] (fp32) for the backward."""
    return (_ext or _load_ext()).forward("sb_attn_fwd_train", False, q, k, v, None, o, m, True, stream)


def sb_attn_fwd_f32(q, k, v, o=None, m=None, want_m=False, stream=None):
    """fp32 forward.  Returns o, or (o, m) when m is given or want_m is set."""
    return (_ext or _load_ext()).forward_f32(q, k, v, o, m, want_m, stream)


def sb_attn_bwd_workspace_bytes(B, H, T, d) -> int:
    return int(load().sb_attn_bwd_workspace_bytes(B, H, T, d))


def sb_attn_bwd(q, k, v, m, dout, dq=None, dk=None, dv=None, workspace=None, stream=None):
    """bf16 backward.  Returns (dq, dk, dv) in fp32."""
    return (_ext or _load_ext()).backward("sb_attn_bwd", False, q, k, v, None, m, dout, dq, dk, dv, None,
                                          workspace, stream)


def sb_attn_fwd_rb(q, k, v, r, o=None, m=None, want_m=True, stream=None):
    """bf16 forward with remainder bias r [H,d] (bf16).  Returns (o, m), or o when want_m is off."""
    if r is None:
        raise SbAttnError("sb_attn_fwd_rb failed: r is required")
    return (_ext or _load_ext()).forward("sb_attn_fwd_rb", False, q, k, v, r, o, m, want_m, stream)


def sb_attn_bwd_rb(q, k, v, r, m, dout, dq=None, dk=None, dv=None, dr=None, workspace=None, stream=None):
    """bf16 backward with remainder bias.  Returns (dq, dk, dv, dr) in fp32; dr is [H,d]."""
    if r is None:
        raise SbAttnError("sb_attn_bwd_rb failed: r is required")
    return (_ext or _load_ext()).backward("sb_attn_bwd_rb", False, q, k, v, r, m, dout, dq, dk, dv, dr,
                                          workspace, stream)


def sb_attn_fwd_gqa(q, k, v, r=None, o=None, m=None, want_m=True, stream=None):
    """bf16 forward with grouped kv heads: q [B,H,T,d], k, v [B,Hkv,T,d]; optional remainder
    bias r [H,d].  Returns (o, m), or o when want_m is off."""
    return (_ext or _load_ext()).forward("sb_attn_fwd_gqa", True, q, k, v, r, o, m, want_m, stream)


def sb_attn_bwd_gqa_workspace_bytes(B, H, Hkv, T, d) -> int:
    """What sb_attn_bwd_gqa allocates itself: with it a far-reaching group's heads are shared out over the chip."""
    return int(load().sb_attn_bwd_gqa_workspace_bytes(B, H, Hkv, T, d))


def sb_attn_bwd_gqa(q, k, v, m, dout, r=None, dq=None, dk=None, dv=None, dr=None, workspace=None, stream=None):
    """bf16 backward with grouped kv heads.  Returns (dq, dk, dv) in fp32 (dk, dv [B,Hkv,T,d]),
    and dr [H,d] as a fourth item when r is given."""
    return (_ext or _load_ext()).backward("sb_attn_bwd_gqa", True, q, k, v, r, m, dout, dq, dk, dv, dr,
                                          workspace, stream)


def sb_attn_varlen_fwd(q, k, v, cu_seqlens, max_T, r=None, o=None, m=None, want_m=True, stream=None):
    """bf16 forward on a packed variable-length batch: q [H,Ttot,d], k, v [Hkv,Ttot,d],
    cu_seqlens int32 [nseq+1] on the GPU, max_T >= the longest sequence.  Returns (o, m) or o."""
    return (_ext or _load_ext()).varlen_forward(q, k, v, cu_seqlens, max_T, r, o, m, want_m, stream)


def sb_attn_varlen_bwd_workspace_bytes(nseq, H, Ttot, max_T, d) -> int:
    return int(load().sb_attn_varlen_bwd_workspace_bytes(nseq, H, Ttot, max_T, d))


def sb_attn_varlen_bwd_gqa_workspace_bytes(nseq, H, Hkv, Ttot, max_T, d) -> int:
    return int(load().sb_attn_varlen_bwd_gqa_workspace_bytes(nseq, H, Hkv, Ttot, max_T, d))


def sb_attn_varlen_bwd(q, k, v, m, dout, cu_seqlens, max_T, r=None, dq=None, dk=None, dv=None, dr=None,
                       workspace=None, stream=None):
    """bf16 backward on a packed variable-length batch.  Returns (dq, dk, dv[, dr]) in fp32."""
    return (_ext or _load_ext()).varlen_backward(q, k, v, m, dout, cu_seqlens, max_T, r, dq, dk, dv, dr,
                                                 workspace, stream)


def sb_attn_decode(q, k, v, T=None, r=None, o=None, m=None, want_m=False, workspace=None, stream=None):
    """Single-token decode: q [B,H,d], cache k, v [B,Hkv,Tcap,d] with the first T rows valid
    (T defaults to Tcap).  Returns o [B,H,d] (bf16), or (o, m) when m is wanted."""
    return (_ext or _load_ext()).decode(q, k, v, T, r, o, m, want_m, workspace, stream, False)


def sb_attn_decode_static(q, k, v, o, T=None, r=None, m=None, stream=None):
    """sb_attn_decode on the library's own static device scratch: nothing is allocated, so the
    caller passes every output (o [B,H,d] bf16, optionally m [B,H] fp32)."""
    return (_ext or _load_ext()).decode(q, k, v, T, r, o, m, False, None, stream, True)


def sb_attn_bwd_dq(q, k, v, m, dout, dq=None, workspace=None, stream=None):
    """Query-stationary pass of the backward.  Returns (dq, workspace)."""
    return (_ext or _load_ext()).backward_dq(q, k, v, m, dout, dq, workspace, stream)


def sb_attn_bwd_dkdv(q, k, v, dout, workspace, dk=None, dv=None, stream=None):
    """Key-stationary pass of the backward (after sb_attn_bwd_dq on the same workspace).  Returns (dk, dv)."""
    return (_ext or _load_ext()).backward_dkdv(q, k, v, dout, workspace, dk, dv, stream)


def sb_diag_mfma_rate(operands, iters=2000, stream=None):
    """MFMA-only rate on the given bf16 operand data.  Returns (TFLOP/s, shader clock in MHz)."""
    if not operands.is_cuda or operands.dtype != torch.bfloat16 or not operands.is_contiguous():
        raise SbAttnError("operands must be a contiguous bf16 tensor on the GPU")
    flop = ctypes.c_double(0.0)
    nbytes = operands.numel() * 2
    with _on(stream):
        ticks = torch.zeros(4, dtype=torch.int64, device=operands.device)
        run = lambda: _check(load().sb_diag_mfma_rate(ctypes.c_void_p(operands.data_ptr()), nbytes, int(iters),
                                                      ctypes.c_void_p(ticks.data_ptr()), ctypes.byref(flop),
                                                      _stream()), "sb_diag_mfma_rate")
        run()
        e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        e0.record()
        run()
        e1.record()
        e1.synchronize()
        ms = e0.elapsed_time(e1)
        t = ticks.cpu().tolist()
    mhz = t[0] / (t[1] / 100e6) / 1e6 if t[1] > 0 else float("nan")
    return flop.value / (ms * 1e-3) / 1e12, mhz


def sb_diag_stream_read(data, iters=10, stream=None):
    """Read bandwidth (GB/s) of a kernel that only loads `data` (any contiguous GPU tensor)."""
    if not data.is_cuda or not data.is_contiguous():
        raise SbAttnError("data must be a contiguous tensor on the GPU")
    nbytes = (data.numel() * data.element_size()) // 16 * 16
    with _on(stream):
        sink = torch.zeros(4, dtype=torch.int32, device=data.device)
        run = lambda: _check(load().sb_diag_stream_read(ctypes.c_void_p(data.data_ptr()), nbytes,
                                                        ctypes.c_void_p(sink.data_ptr()), _stream()),
                             "sb_diag_stream_read")
        for _ in range(2):
            run()
        e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        e0.record()
        for _ in range(iters):
            run()
        e1.record()
        e1.synchronize()
    return nbytes * iters / (e0.elapsed_time(e1) * 1e-3) / 1e9


def sb_diag_fwd_clock(q, k, v, o, m, stream=None):
    """sb_attn_fwd_train that also returns the shader clock (MHz) its first workgroup saw."""
    B, H, T, d = _dims(q)
    with _on(stream):
        clocks = torch.zeros(4, dtype=torch.int64, device=q.device)
        rc = load().sb_diag_fwd_clock(_ptr(q, torch.bfloat16, None, "q"), _ptr(k, torch.bfloat16, q.shape, "k"),
                                      _ptr(v, torch.bfloat16, q.shape, "v"), _ptr(o, torch.bfloat16, q.shape, "o"),
                                      _ptr(m, torch.float32, (B, H, T), "m"), B, H, T, d,
                                      ctypes.c_void_p(clocks.data_ptr()), _stream())
        _check(rc, "sb_diag_fwd_clock")
        c = clocks.cpu().tolist()
    ref = c[3] - c[1]
    return (c[2] - c[0]) / (ref / 100e6) / 1e6 if ref > 0 else float("nan")


def sb_diag_fwd_tri(q, k, v, o=None, m=None, stream=None):
    """Training forward with the in-tile cumulative sum taken by triangular MFMA (d = 128)."""
    B, H, T, d = _dims(q)
    inputs = [_ptr(t, torch.bfloat16, q.shape, name) for t, name in ((q, "q"), (k, "k"), (v, "v"))]
    current = torch.cuda.current_stream()
    with _on(stream):
        if o is None:
            o = torch.empty_like(q)
            o.record_stream(current)
        if m is None:
            m = torch.empty((B, H, T), dtype=torch.float32, device=q.device)
            m.record_stream(current)
        rc = load().sb_diag_fwd_tri(*inputs, _ptr(o, torch.bfloat16, q.shape, "o"),
                                    _ptr(m, torch.float32, (B, H, T), "m"), B, H, T, d, _stream())
    _check(rc, "sb_diag_fwd_tri")
    return o, m
