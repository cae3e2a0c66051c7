"""Thin Python binding of libomnitide.so (argument marshalling only).

Each function has the name of the C entry point it calls, takes torch tensors where the C
function takes device pointers, checks dtype / device / contiguity / shape, passes the current
HIP stream, and raises ``OmnitideError`` with the library's status code on failure.  Every step
of the computation runs in the HIP kernels; nothing here computes.  If the library has not been
built the first call raises (there is no fallback).

Tensor dtypes: unsigned 64-bit outputs (unit_wsum, unit_score) are held in torch.int64 tensors
and unsigned 32-bit flags in torch.int32 tensors (same bits; all values fit the signed range).
"""
from __future__ import annotations

import ctypes
import os
from typing import Optional, Sequence

import torch

_PKG = os.path.dirname(os.path.abspath(__file__))
LIB_PATH = os.path.join(_PKG, "libomnitide.so")

OK, E_NULL, E_SHAPE, E_DTYPE, E_WEIGHT, E_CAPACITY, E_WORKSPACE, E_ALIAS, E_HIP, E_SCRATCH = \
    0, -1, -2, -3, -4, -5, -6, -7, -8, -9
NOALLOC_SCRATCH_BYTES = 64 << 20
E_BUDGET, E_TAGS, E_RANGE = -16, -17, -18
BF16, F32 = 0, 1
ROPE_HALF, ROPE_INTERLEAVED = 0, 1

EXPORTS = ("omnitide_score_units", "omnitide_select_units", "omnitide_compact_kv",
           "omnitide_compact_kv_rope", "omnitide_plan_spans",
           "omnitide_plan_spans_workspace_bytes", "omnitide_compact_kv_spans",
           "omnitide_compact_workspace_bytes", "omnitide_chunk_attn",
           "omnitide_chunk_attn_noalloc",
           "omnitide_attn_workspace_bytes", "omnitide_span_attn", "omnitide_evict_native",
           "omnitide_evict_native_workspace_bytes", "omnitide_evict_native_rope",
           "omnitide_evict_native_rope_workspace_bytes", "omnitide_pack_suffix",
           "omnitide_pack_suffix_workspace_bytes", "omnitide_place_chunk",
           "omnitide_place_chunk_workspace_bytes",
           "omnitide_span_attn_workspace_bytes", "omnitide_decode_attn",
           "omnitide_decode_workspace_bytes", "omnitide_decode_span_attn",
           "omnitide_decode_span_workspace_bytes", "omnitide_status_string", "omnitide_version")


class OmnitideError(RuntimeError):
    def __init__(self, code: int, where: str):
        self.code = code
        super().__init__(f"{where}: {status_string(code)} (status {code})")


_lib = None

_P = ctypes.c_void_p
_I = ctypes.c_int
_SZ = ctypes.c_size_t


def lib() -> ctypes.CDLL:
    """The loaded HIP library; raises if it has not been built."""
    global _lib
    if _lib is None:
        if not os.path.exists(LIB_PATH):
            raise RuntimeError(f"{LIB_PATH} is missing: build it with "
                               "`python -m paper_2609_34653_amd.build` (hipcc, gfx950)")
        L = ctypes.CDLL(LIB_PATH)
        L.omnitide_score_units.argtypes = [_P, _I, _I, _I, _I, _I, _P, _P, _P, _I, _P, _P, _P,
                                           _P, _P, _P, _P]
        L.omnitide_select_units.argtypes = [_P, _P, _P, _P, _P, _I, _I, _I, _I, _P, _P, _P, _P,
                                            _P]
        L.omnitide_compact_kv.argtypes = [_P, _P, _I, _I, _I, _I, _I, _I, _P, _P, _P, _P, _P, _P,
                                          _I, _P, _P, _P, _P, _I, _P, _P, _I, _P, _P, _P, _P, _P,
                                          _P, _P, _P, _SZ, _P, _P]
        L.omnitide_compact_kv_rope.argtypes = (L.omnitide_compact_kv.argtypes[:-2] +
                                               [ctypes.c_double, _I, _I, _P, _P])
        L.omnitide_compact_kv_spans.argtypes = L.omnitide_compact_kv_rope.argtypes
        L.omnitide_plan_spans.argtypes = [_P, _P, _P, _P, _P, _P, _I, _I, _I, _I, _I, _I, _I,
                                          _I, _I, _P, _P, _P, _P, _SZ, _P, _P]
        L.omnitide_plan_spans_workspace_bytes.argtypes = [_I, _I, _I]
        L.omnitide_plan_spans_workspace_bytes.restype = _SZ
        L.omnitide_compact_workspace_bytes.argtypes = [_I, _I, _I]
        L.omnitide_compact_workspace_bytes.restype = _SZ
        L.omnitide_chunk_attn.argtypes = [_P, _P, _P, _I, _P, _I, _I, _I, _I, _I, _I,
                                          ctypes.c_float, _P, _I, _P, _SZ, _P, _P]
        L.omnitide_chunk_attn_noalloc.argtypes = [_P, _P, _P, _P, _I, _I, _I, _I, _I, _I,
                                                  ctypes.c_float, _P, _I, _P, _P]
        L.omnitide_attn_workspace_bytes.argtypes = [_I, _I, _I, _I, _I, _I, _I]
        L.omnitide_attn_workspace_bytes.restype = _SZ
        L.omnitide_span_attn.argtypes = [_P, _P, _P, _P, _P, _P, _I, _I, _I, _I, _I, _I,
                                         ctypes.c_float, _I, _P, _P, _SZ, _P, _P]
        L.omnitide_span_attn_workspace_bytes.argtypes = [_I, _I, _I, _I, _I, _I]
        L.omnitide_span_attn_workspace_bytes.restype = _SZ
        L.omnitide_evict_native.argtypes = [_I, _I, _P, _P, _P, _P, _P, _I, _P, _P, _P, _P, _P,
                                            _SZ, _P, _P]
        L.omnitide_evict_native_workspace_bytes.argtypes = [_I, _I]
        L.omnitide_evict_native_workspace_bytes.restype = _SZ
        L.omnitide_evict_native_rope.argtypes = [_I, _I, _P, _P, _P, _P, _P, _I, _P, _I, _I, _I,
                                                 ctypes.c_double, _I, _I, _P, _P, _P, _P, _P,
                                                 _SZ, _P, _P]
        L.omnitide_evict_native_rope_workspace_bytes.argtypes = [_I, _I, _I]
        L.omnitide_evict_native_rope_workspace_bytes.restype = _SZ
        L.omnitide_pack_suffix.argtypes = [_P, _P, _I, _I, _I, _I, _I, _I, _I, _P, _P, _P, _P,
                                           _P, _P, _P, _SZ, _P]
        L.omnitide_pack_suffix_workspace_bytes.argtypes = [_I, _I, _I, _I, _I]
        L.omnitide_pack_suffix_workspace_bytes.restype = _SZ
        L.omnitide_place_chunk.argtypes = [_P, _P, _I, _I, _I, _I, _I, _P, _P, _P, _P, _P, _P,
                                           _P, _I, _P, _P, _P, _P, _P, _SZ, _P, _P]
        L.omnitide_place_chunk_workspace_bytes.argtypes = [_I, _I]
        L.omnitide_place_chunk_workspace_bytes.restype = _SZ
        L.omnitide_decode_attn.argtypes = [_P, _P, _P, _P, _I, _I, _I, _I, _I, _I,
                                           ctypes.c_float, _P, _P, _SZ, _P, _P]
        L.omnitide_decode_workspace_bytes.argtypes = [_I, _I, _I, _I, _I, _I]
        L.omnitide_decode_workspace_bytes.restype = _SZ
        L.omnitide_decode_span_attn.argtypes = L.omnitide_span_attn.argtypes
        L.omnitide_decode_span_workspace_bytes.argtypes = [_I, _I, _I, _I, _I, _I]
        L.omnitide_decode_span_workspace_bytes.restype = _SZ
        L.omnitide_status_string.argtypes = [_I]
        L.omnitide_status_string.restype = ctypes.c_char_p
        L.omnitide_version.restype = ctypes.c_char_p
        for name in ("omnitide_score_units", "omnitide_select_units", "omnitide_compact_kv",
                     "omnitide_compact_kv_rope", "omnitide_compact_kv_spans",
                     "omnitide_plan_spans", "omnitide_chunk_attn",
                     "omnitide_chunk_attn_noalloc", "omnitide_span_attn",
                     "omnitide_evict_native", "omnitide_evict_native_rope",
                     "omnitide_pack_suffix", "omnitide_place_chunk",
                     "omnitide_decode_attn", "omnitide_decode_span_attn"):
            getattr(L, name).restype = _I
        _lib = L
    return _lib


def status_string(code: int) -> str:
    return lib().omnitide_status_string(int(code)).decode()


def version() -> str:
    return lib().omnitide_version().decode()


# ----------------------------------------------------------------------------- marshalling

# A call checks and passes up to 30 tensors, so the common case (a plain contiguous device tensor of
# the right type and size) takes one short function per tensor that returns the address; anything
# else goes through _need, which raises or accepts it.  Four calls' marshalling bounds a small step:
# the 1.6K-token float32 step took 64 us with separate checks and pointer objects, 49 us so.

def _stream(stream) -> Optional[int]:
    if stream is None:
        return torch._C._cuda_getCurrentRawStream(torch.cuda.current_device())
    return stream.cuda_stream if hasattr(stream, "cuda_stream") else stream


def _need(t: torch.Tensor, name: str, dtypes: Sequence[torch.dtype], numel: Optional[int] = None):
    if not isinstance(t, torch.Tensor):
        raise TypeError(f"{name} must be a tensor")
    if t.dtype not in dtypes:
        raise TypeError(f"{name}: dtype {t.dtype} not in {list(dtypes)}")
    if not t.is_cuda:
        raise ValueError(f"{name} must be a device tensor")
    if not t.is_contiguous():
        raise ValueError(f"{name} must be contiguous")
    if numel is not None and t.numel() != numel:
        raise ValueError(f"{name}: expected {numel} elements, got {t.numel()}")


def _check(code: int, where: str):
    if code != OK:
        raise OmnitideError(code, where)


_T, _BF16, _F32, _I32, _I64, _U8 = (torch.Tensor, torch.bfloat16, torch.float32, torch.int32,
                                    torch.int64, torch.uint8)


def _dev(t, name: str, dtype: torch.dtype, numel: int) -> int:
    """Address of a contiguous device tensor of `dtype` and `numel` elements."""
    if not (type(t) is _T and t.dtype is dtype and t.is_cuda and t.is_contiguous()
            and t.numel() == numel):
        _need(t, name, (dtype,), numel)
    return t.data_ptr()


def _buf(t, name: str = "workspace") -> int:
    """Address of a uint8 device buffer of any size."""
    if not (type(t) is _T and t.dtype is _U8 and t.is_cuda and t.is_contiguous()):
        _need(t, name, (_U8,))
    return t.data_ptr()


def _pool(t, name: str) -> int:
    """Address of a bf16 or float32 device tensor."""
    if not (type(t) is _T and (t.dtype is _BF16 or t.dtype is _F32) and t.is_cuda
            and t.is_contiguous()):
        _need(t, name, (_BF16, _F32))
    return t.data_ptr()


def _status(t) -> Optional[int]:
    return None if t is None else _dev(t, "d_status", _I32, 1)


def _pool_dims(t: torch.Tensor, name: str):
    """[n_seg, n_slots, H, d] (or [n_slots, H, d] = one segment)."""
    if t.dim() == 3:
        return 1, t.shape[0], t.shape[1], t.shape[2]
    if t.dim() == 4:
        return tuple(t.shape)
    raise ValueError(f"{name} must be [n_seg, n_slots, H, d] or [n_slots, H, d]")


def _kv_dtype(t: torch.Tensor) -> int:
    return BF16 if t.dtype == torch.bfloat16 else F32


_F4 = ctypes.c_float * 4


def omnitide_score_units(k, unit_id, modality, weights, n_units, unit_wsum, unit_len,
                         unit_first_slot, unit_last_slot, unit_flags, d_status=None, stream=None):
    n_seg, n_slots, H, d = _pool_dims(k, "k")
    ns, nu = n_seg * n_slots, n_seg * n_units
    args = (_pool(k, "k"), _kv_dtype(k), n_seg, n_slots, H, d, _dev(unit_id, "unit_id", _I32, ns),
            _dev(modality, "modality", _U8, ns), _F4(*[float(x) for x in weights]), n_units,
            _dev(unit_wsum, "unit_wsum", _I64, nu), _dev(unit_len, "unit_len", _I32, nu),
            _dev(unit_first_slot, "unit_first_slot", _I32, nu),
            _dev(unit_last_slot, "unit_last_slot", _I32, nu),
            _dev(unit_flags, "unit_flags", _I32, nu), _status(d_status))
    _check(lib().omnitide_score_units(*args, _stream(stream)), "omnitide_score_units")


def omnitide_select_units(unit_wsum, unit_len, unit_first_slot, unit_last_slot, unit_flags,
                          n_seg, n_units, budget_tokens, recent_tokens, unit_score, keep,
                          kept_tokens, d_status=None, stream=None):
    nu = n_seg * n_units
    args = (_dev(unit_wsum, "unit_wsum", _I64, nu), _dev(unit_len, "unit_len", _I32, nu),
            _dev(unit_first_slot, "unit_first_slot", _I32, nu),
            _dev(unit_last_slot, "unit_last_slot", _I32, nu),
            _dev(unit_flags, "unit_flags", _I32, nu), n_seg, n_units, budget_tokens,
            recent_tokens, _dev(unit_score, "unit_score", _I64, nu), _dev(keep, "keep", _U8, nu),
            _dev(kept_tokens, "kept_tokens", _I32, n_seg), _status(d_status))
    _check(lib().omnitide_select_units(*args, _stream(stream)), "omnitide_select_units")


def omnitide_plan_spans_workspace_bytes(n_seg, n_slots, n_units) -> int:
    return int(lib().omnitide_plan_spans_workspace_bytes(n_seg, n_slots, n_units))


def omnitide_plan_spans(unit_len, unit_first_slot, unit_last_slot, unit_flags, unit_id, modality,
                        n_seg, n_slots, n_units, low_watermark, high_watermark, recent_tokens,
                        sink_video, sink_audio, text_budget, keep_len, keep_slot, kept_tokens,
                        workspace, d_status=None, stream=None):
    nu, ns = n_seg * n_units, n_seg * n_slots
    args = (_dev(unit_len, "unit_len", _I32, nu),
            _dev(unit_first_slot, "unit_first_slot", _I32, nu),
            _dev(unit_last_slot, "unit_last_slot", _I32, nu),
            _dev(unit_flags, "unit_flags", _I32, nu), _dev(unit_id, "unit_id", _I32, ns),
            _dev(modality, "modality", _U8, ns), n_seg, n_slots, n_units, low_watermark,
            high_watermark, recent_tokens, sink_video, sink_audio, text_budget,
            _dev(keep_len, "keep_len", _I32, nu), _dev(keep_slot, "keep_slot", _U8, ns),
            _dev(kept_tokens, "kept_tokens", _I32, n_seg), _buf(workspace), workspace.numel(),
            _status(d_status))
    _check(lib().omnitide_plan_spans(*args, _stream(stream)), "omnitide_plan_spans")


def omnitide_compact_workspace_bytes(n_seg, n_units, cap_dst) -> int:
    return int(lib().omnitide_compact_workspace_bytes(n_seg, n_units, cap_dst))


def _compact_call_args(k_src, v_src, page_size, unit_id_src, modality_src, pos_src, keep,
                       unit_len, unit_first_slot, n_units, k_chunk, v_chunk, chunk_modality,
                       chunk_unit, k_dst, v_dst, unit_id_dst, modality_dst, pos_dst, src_of_dst,
                       unit_remap, n_ctx, n_pages, workspace, d_status, per_slot=False):
    """Checked C arguments shared by the compaction entry points (all but the rotary arguments,
    the status and the stream).  `keep` is the uint8 keep flags per unit, or (per_slot) the span
    plan's uint8 keep mask per slot."""
    n_seg, n_slots, H, d = _pool_dims(k_src, "k_src")
    dt = k_src.dtype
    ks = _pool(k_src, "k_src")
    vs = _dev(v_src, "v_src", dt, k_src.numel())
    ns, nu = n_seg * n_slots, n_seg * n_units
    src = (_dev(unit_id_src, "unit_id_src", _I32, ns), _dev(modality_src, "modality_src", _U8, ns),
           _dev(pos_src, "pos_src", _I32, ns),
           _dev(keep, "keep_slot", _U8, ns) if per_slot else _dev(keep, "keep", _U8, nu),
           _dev(unit_len, "unit_len", _I32, nu),
           _dev(unit_first_slot, "unit_first_slot", _I32, nu))
    L = 0 if chunk_modality is None else chunk_modality.numel()
    if L:
        nc = n_seg * L * H * d
        chunk = (_dev(k_chunk, "k_chunk", dt, nc), _dev(v_chunk, "v_chunk", dt, nc),
                 _dev(chunk_modality, "chunk_modality", _U8, L),
                 _dev(chunk_unit, "chunk_unit", _I32, L))
    else:
        chunk = tuple(None if t is None else t.data_ptr()
                      for t in (k_chunk, v_chunk, chunk_modality, chunk_unit))
    ds, cap, Hd, dd = _pool_dims(k_dst, "k_dst")
    if ds != n_seg or Hd != H or dd != d:
        raise ValueError("k_dst shape does not match k_src")
    nd = n_seg * cap
    if k_dst.dtype is not dt or not k_dst.is_cuda or not k_dst.is_contiguous():
        _need(k_dst, "k_dst", (dt,))
    return (ks, vs, _kv_dtype(k_src), n_seg, n_slots, H, d, page_size, *src, n_units, *chunk, L,
            k_dst.data_ptr(), _dev(v_dst, "v_dst", dt, k_dst.numel()), cap,
            _dev(unit_id_dst, "unit_id_dst", _I32, nd),
            _dev(modality_dst, "modality_dst", _U8, nd), _dev(pos_dst, "pos_dst", _I32, nd),
            _dev(src_of_dst, "src_of_dst", _I32, nd), _dev(unit_remap, "unit_remap", _I32, nu),
            _dev(n_ctx, "n_ctx", _I32, n_seg), _dev(n_pages, "n_pages", _I32, n_seg),
            _buf(workspace), workspace.numel())


def omnitide_compact_kv(k_src, v_src, page_size, unit_id_src, modality_src, pos_src, keep,
                        unit_len, unit_first_slot, n_units, k_chunk, v_chunk, chunk_modality,
                        chunk_unit, k_dst, v_dst, unit_id_dst, modality_dst, pos_dst, src_of_dst,
                        unit_remap, n_ctx, n_pages, workspace, d_status=None, stream=None):
    args = _compact_call_args(k_src, v_src, page_size, unit_id_src, modality_src, pos_src, keep,
                              unit_len, unit_first_slot, n_units, k_chunk, v_chunk,
                              chunk_modality, chunk_unit, k_dst, v_dst, unit_id_dst,
                              modality_dst, pos_dst, src_of_dst, unit_remap, n_ctx, n_pages,
                              workspace, d_status)
    _check(lib().omnitide_compact_kv(*args, _status(d_status), _stream(stream)),
           "omnitide_compact_kv")


def omnitide_compact_kv_rope(k_src, v_src, page_size, unit_id_src, modality_src, pos_src, keep,
                             unit_len, unit_first_slot, n_units, k_chunk, v_chunk,
                             chunk_modality, chunk_unit, k_dst, v_dst, unit_id_dst,
                             modality_dst, pos_dst, src_of_dst, unit_remap, n_ctx, n_pages,
                             workspace, rope_base, rope_dims, rope_style=ROPE_HALF,
                             d_status=None, stream=None):
    args = _compact_call_args(k_src, v_src, page_size, unit_id_src, modality_src, pos_src, keep,
                              unit_len, unit_first_slot, n_units, k_chunk, v_chunk,
                              chunk_modality, chunk_unit, k_dst, v_dst, unit_id_dst,
                              modality_dst, pos_dst, src_of_dst, unit_remap, n_ctx, n_pages,
                              workspace, d_status)
    _check(lib().omnitide_compact_kv_rope(*args, float(rope_base), int(rope_dims),
                                          int(rope_style), _status(d_status), _stream(stream)),
           "omnitide_compact_kv_rope")


def omnitide_compact_kv_spans(k_src, v_src, page_size, unit_id_src, modality_src, pos_src,
                              keep_slot, unit_len, unit_first_slot, n_units, k_chunk, v_chunk,
                              chunk_modality, chunk_unit, k_dst, v_dst, unit_id_dst,
                              modality_dst, pos_dst, src_of_dst, unit_remap, n_ctx, n_pages,
                              workspace, rope_base=0.0, rope_dims=0, rope_style=ROPE_HALF,
                              d_status=None, stream=None):
    args = _compact_call_args(k_src, v_src, page_size, unit_id_src, modality_src, pos_src,
                              keep_slot, unit_len, unit_first_slot, n_units, k_chunk, v_chunk,
                              chunk_modality, chunk_unit, k_dst, v_dst, unit_id_dst,
                              modality_dst, pos_dst, src_of_dst, unit_remap, n_ctx, n_pages,
                              workspace, d_status, per_slot=True)
    _check(lib().omnitide_compact_kv_spans(*args, float(rope_base), int(rope_dims),
                                           int(rope_style), _status(d_status), _stream(stream)),
           "omnitide_compact_kv_spans")


def omnitide_attn_workspace_bytes(n_seg, cap, chunk_len, n_q_heads, n_kv_heads, head_dim,
                                  dtype=BF16) -> int:
    return int(lib().omnitide_attn_workspace_bytes(dtype, n_seg, cap, chunk_len, n_q_heads,
                                                   n_kv_heads, head_dim))


def _q_dims(q, k):
    """(n_seg, tokens, query heads, d, cap, KV heads) of q [n_seg, L, Hq, d] (or [L, Hq, d]) and
    its pool."""
    if q.dim() == 3:
        n_seg, (L, Hq, d) = 1, q.shape
    else:
        n_seg, L, Hq, d = q.shape
    ds, cap, Hkv, dd = _pool_dims(k, "k")
    if ds != n_seg or dd != d:
        raise ValueError("k shape does not match q")
    return n_seg, L, Hq, d, cap, Hkv


def _out(out, numel) -> int:
    """Address of a float32 or bf16 output."""
    if not (type(out) is _T and (out.dtype is _F32 or out.dtype is _BF16) and out.is_cuda
            and out.is_contiguous() and out.numel() == numel):
        _need(out, "out", (_F32, _BF16), numel)
    return out.data_ptr()


def omnitide_chunk_attn(q, k, v, n_ctx, scale, out, workspace=None, d_status=None, stream=None):
    """q/k/v bf16 or float32 (all the same); out float32 or bf16 (its dtype selects)."""
    n_seg, L, Hq, d, cap, Hkv = _q_dims(q, k)
    args = (_pool(q, "q"), _dev(k, "k", q.dtype, k.numel()), _dev(v, "v", q.dtype, k.numel()),
            _kv_dtype(q), _dev(n_ctx, "n_ctx", _I32, n_seg), n_seg, cap, L, Hq, Hkv, d,
            float(scale), _out(out, q.numel()), _kv_dtype(out),
            None if workspace is None else _buf(workspace),
            0 if workspace is None else workspace.numel(), _status(d_status))
    _check(lib().omnitide_chunk_attn(*args, _stream(stream)), "omnitide_chunk_attn")


def omnitide_chunk_attn_noalloc(q, k, v, n_ctx, scale, out, d_status=None, stream=None):
    """omnitide_chunk_attn with the library's fixed scratch (allocates nothing)."""
    n_seg, L, Hq, d, cap, Hkv = _q_dims(q, k)
    args = (_dev(q, "q", _BF16, q.numel()), _dev(k, "k", _BF16, k.numel()),
            _dev(v, "v", _BF16, k.numel()), _dev(n_ctx, "n_ctx", _I32, n_seg), n_seg, cap, L, Hq,
            Hkv, d, float(scale), _out(out, q.numel()), _kv_dtype(out), _status(d_status))
    _check(lib().omnitide_chunk_attn_noalloc(*args, _stream(stream)),
           "omnitide_chunk_attn_noalloc")


def omnitide_span_attn_workspace_bytes(n_seg, cap, chunk_len, n_q_heads, n_kv_heads,
                                       head_dim) -> int:
    return int(lib().omnitide_span_attn_workspace_bytes(n_seg, cap, chunk_len, n_q_heads,
                                                        n_kv_heads, head_dim))


def _span_call_args(q, k, v, key_pos, span, q_pos0, scale, out, workspace, d_status,
                    skip_empty_tiles, position_order):
    """Checked C arguments of the two calls over a pool with holes (all but the stream)."""
    n_seg, L, Hq, d, cap, Hkv = _q_dims(q, k)
    return (_dev(q, "q", _BF16, q.numel()), _dev(k, "k", _BF16, k.numel()),
            _dev(v, "v", _BF16, k.numel()), _dev(key_pos, "key_pos", _I32, n_seg * cap),
            _dev(span, "span", _I32, n_seg), _dev(q_pos0, "q_pos0", _I32, n_seg), n_seg, cap, L,
            Hq, Hkv, d, float(scale), 2 if position_order else 1 if skip_empty_tiles else 0,
            _dev(out, "out", _F32, q.numel()), _buf(workspace), workspace.numel(),
            _status(d_status))


def omnitide_span_attn(q, k, v, key_pos, span, q_pos0, scale, out, workspace, d_status=None,
                       stream=None, skip_empty_tiles=True, position_order=False):
    """q [n_seg, L, Hq, d] bf16; k/v [n_seg, cap, Hkv, d] bf16; key_pos int32 [n_seg * cap]
    (-1 = empty slot); span, q_pos0 int32 [n_seg] (device); out float32 like q.
    Traversal: position_order (the entries gathered in position order; they must hold the
    positions 0 .. q_pos0 + L - 1 once each), else tile skipping if skip_empty_tiles, else the
    full span."""
    args = _span_call_args(q, k, v, key_pos, span, q_pos0, scale, out, workspace, d_status,
                           skip_empty_tiles, position_order)
    _check(lib().omnitide_span_attn(*args, _stream(stream)), "omnitide_span_attn")


def omnitide_decode_span_workspace_bytes(n_seg, cap, n_q, n_q_heads, n_kv_heads,
                                         head_dim) -> int:
    return int(lib().omnitide_decode_span_workspace_bytes(n_seg, cap, n_q, n_q_heads, n_kv_heads,
                                                          head_dim))


def omnitide_decode_span_attn(q, k, v, key_pos, span, q_pos0, scale, out, workspace,
                              d_status=None, stream=None, skip_empty_tiles=True,
                              position_order=False):
    """Decode attention of n_q tokens over a pool with holes: q [n_seg, n_q, Hq, d] bf16;
    k/v [n_seg, cap, Hkv, d] bf16; key_pos int32 [n_seg * cap] (-1 = empty slot); span, q_pos0
    int32 [n_seg] (device); out float32 like q.  Traversal as omnitide_span_attn."""
    args = _span_call_args(q, k, v, key_pos, span, q_pos0, scale, out, workspace, d_status,
                           skip_empty_tiles, position_order)
    _check(lib().omnitide_decode_span_attn(*args, _stream(stream)), "omnitide_decode_span_attn")


def omnitide_evict_native_workspace_bytes(n_seg, n_units) -> int:
    return int(lib().omnitide_evict_native_workspace_bytes(n_seg, n_units))


def _evict_call_args(unit_id, pos, n_seg, n_units, unit_len, keep, keep_len):
    """Checked (unit_id, pos, keep, keep_len, unit_len) addresses and cap of an eviction."""
    cap = unit_id.numel() // n_seg
    nu = n_seg * n_units
    head = (_dev(unit_id, "unit_id", _I32, n_seg * cap), _dev(pos, "pos", _I32, n_seg * cap))
    if keep_len is not None:
        plan = (None, _dev(keep_len, "keep_len", _I32, nu))
    else:
        plan = (_dev(keep, "keep", _U8, nu), None)
    return cap, nu, (*head, *plan, _dev(unit_len, "unit_len", _I32, nu))


def omnitide_evict_native(unit_id, pos, n_seg, n_units, unit_len, unit_remap, kept_tokens,
                          n_kept_units, span, workspace, keep=None, keep_len=None,
                          d_status=None, stream=None):
    """Logical eviction in place of the tags unit_id / pos ([n_seg * cap] int32)."""
    cap, nu, head = _evict_call_args(unit_id, pos, n_seg, n_units, unit_len, keep, keep_len)
    args = (n_seg, cap, *head, n_units, _dev(unit_remap, "unit_remap", _I32, nu),
            _dev(kept_tokens, "kept_tokens", _I32, n_seg),
            _dev(n_kept_units, "n_kept_units", _I32, n_seg), _dev(span, "span", _I32, n_seg),
            _buf(workspace), workspace.numel(), _status(d_status))
    _check(lib().omnitide_evict_native(*args, _stream(stream)), "omnitide_evict_native")


def omnitide_evict_native_rope_workspace_bytes(n_seg, n_units, cap) -> int:
    return int(lib().omnitide_evict_native_rope_workspace_bytes(n_seg, n_units, cap))


def omnitide_evict_native_rope(unit_id, pos, k, n_seg, n_units, unit_len, unit_remap,
                               kept_tokens, n_kept_units, span, workspace, rope_base, rope_dims,
                               rope_style=ROPE_HALF, keep=None, keep_len=None, d_status=None,
                               stream=None):
    """Logical eviction in place plus the rotary adjustment, in place, of the keys k
    ([n_seg, cap, H, d] bf16 or float32) whose positions shift."""
    ds, kcap, H, d = _pool_dims(k, "k")
    if ds != n_seg or kcap != unit_id.numel() // n_seg:
        raise ValueError("k shape does not match the tags")
    kp = _pool(k, "k")
    cap, nu, head = _evict_call_args(unit_id, pos, n_seg, n_units, unit_len, keep, keep_len)
    args = (n_seg, cap, *head, n_units, kp, _kv_dtype(k), H, d, float(rope_base), int(rope_dims),
            int(rope_style), _dev(unit_remap, "unit_remap", _I32, nu),
            _dev(kept_tokens, "kept_tokens", _I32, n_seg),
            _dev(n_kept_units, "n_kept_units", _I32, n_seg), _dev(span, "span", _I32, n_seg),
            _buf(workspace), workspace.numel(), _status(d_status))
    _check(lib().omnitide_evict_native_rope(*args, _stream(stream)),
           "omnitide_evict_native_rope")


def omnitide_pack_suffix_workspace_bytes(dtype, n_seg, cap, n_kv_heads, head_dim) -> int:
    return int(lib().omnitide_pack_suffix_workspace_bytes(dtype, n_seg, cap, n_kv_heads,
                                                          head_dim))


def omnitide_pack_suffix(k, v, page_size, min_pages, unit_id, modality, pos, span, cut, moved,
                         workspace, stream=None):
    """Ordered-suffix packing in place of pools k/v [n_seg, cap, H, d] and their tags."""
    n_seg, cap, H, d = _pool_dims(k, "k")
    ns = n_seg * cap
    args = (_pool(k, "k"), _dev(v, "v", k.dtype, k.numel()), _kv_dtype(k), n_seg, cap, H, d,
            page_size, min_pages, _dev(unit_id, "unit_id", _I32, ns),
            _dev(modality, "modality", _U8, ns), _dev(pos, "pos", _I32, ns),
            _dev(span, "span", _I32, n_seg), _dev(cut, "cut", _I32, n_seg),
            _dev(moved, "moved", _I32, n_seg), _buf(workspace), workspace.numel())
    _check(lib().omnitide_pack_suffix(*args, _stream(stream)), "omnitide_pack_suffix")


def omnitide_place_chunk_workspace_bytes(n_seg, cap) -> int:
    return int(lib().omnitide_place_chunk_workspace_bytes(n_seg, cap))


def omnitide_place_chunk(k, v, unit_id, modality, pos, k_chunk, v_chunk, chunk_modality,
                         chunk_unit, kept_tokens, n_kept_units, chunk_slot, span, workspace,
                         d_status=None, stream=None):
    """The chunk into the lowest run of empty slots of pools k/v [n_seg, cap, H, d]."""
    n_seg, cap, H, d = _pool_dims(k, "k")
    L = chunk_modality.numel()
    ns, nc, dt = n_seg * cap, n_seg * L * H * d, k.dtype
    args = (_pool(k, "k"), _dev(v, "v", dt, k.numel()), _kv_dtype(k), n_seg, cap, H, d,
            _dev(unit_id, "unit_id", _I32, ns), _dev(modality, "modality", _U8, ns),
            _dev(pos, "pos", _I32, ns), _dev(k_chunk, "k_chunk", dt, nc),
            _dev(v_chunk, "v_chunk", dt, nc), _dev(chunk_modality, "chunk_modality", _U8, L),
            _dev(chunk_unit, "chunk_unit", _I32, L), L,
            _dev(kept_tokens, "kept_tokens", _I32, n_seg),
            _dev(n_kept_units, "n_kept_units", _I32, n_seg),
            _dev(chunk_slot, "chunk_slot", _I32, n_seg), _dev(span, "span", _I32, n_seg),
            _buf(workspace), workspace.numel(), _status(d_status))
    _check(lib().omnitide_place_chunk(*args, _stream(stream)), "omnitide_place_chunk")


def omnitide_decode_workspace_bytes(n_seg, cap, n_q, n_q_heads, n_kv_heads, head_dim) -> int:
    return int(lib().omnitide_decode_workspace_bytes(n_seg, cap, n_q, n_q_heads, n_kv_heads,
                                                     head_dim))


def omnitide_decode_attn(q, k, v, n_ctx, scale, out, workspace=None, d_status=None,
                         stream=None):
    """q [n_seg, n_q, Hq, d] bf16 (the last n_q tokens), k/v [n_seg, cap, Hkv, d] bf16,
    n_ctx int32 [n_seg] (device), out float32 like q."""
    if q.dim() == 3:
        q = q.unsqueeze(0)
    n_seg, n_q, Hq, d = q.shape
    ns, cap, Hkv, dk = _pool_dims(k, "k")
    if ns != n_seg or dk != d:
        raise ValueError("k does not match q")
    args = (_dev(q, "q", _BF16, q.numel()), _dev(k, "k", _BF16, k.numel()),
            _dev(v, "v", _BF16, k.numel()), _dev(n_ctx, "n_ctx", _I32, n_seg), n_seg, cap, n_q,
            Hq, Hkv, d, float(scale), _dev(out, "out", _F32, q.numel()),
            None if workspace is None else _buf(workspace),
            0 if workspace is None else workspace.numel(), _status(d_status))
    _check(lib().omnitide_decode_attn(*args, _stream(stream)), "omnitide_decode_attn")
