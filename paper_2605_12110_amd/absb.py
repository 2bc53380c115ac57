"""Thin Python binding of libabsb.so: same names as the C ABI, argument marshalling only.

Every step of the path runs in the library's HIP kernels; this module converts torch
tensors to device pointers, keeps the host-side arrays alive and turns status codes into
exceptions.  There is no fallback: a missing library or a missing GPU raises.
"""
from __future__ import annotations

import ctypes as C
import os
import threading
from dataclasses import dataclass
from typing import Optional, Sequence

import numpy as np

_HERE = os.path.dirname(os.path.abspath(__file__))
# ABSB_LIB names another build of the same library (the host-sanitizer build of tests/sanitized.py)
LIB_PATH = os.environ.get("ABSB_LIB") or os.path.join(_HERE, "libabsb.so")

F16, BF16 = 0, 1
REPR_MEAN, REPR_MINMAX = 0, 1
SELECT_GROUP, SELECT_PER_QUERY_HEAD, SELECT_GROUP_MAX = 0, 1, 2
STEP_AUTO, STEP_PIPELINED, STEP_UNITS, STEP_PER_STAGE = 0, 1, 2, 3

OK, ERR_NULL, ERR_BAD_SHAPE, ERR_BAD_BLOCK_SIZE, ERR_UNSUPPORTED, ERR_WORKSPACE, ERR_HIP = 0, -1, -2, -3, -4, -5, -6
ERR_STATIC_WORKSPACE = -7
STATIC_WORKSPACE_BYTES = 16 << 20

EXPORTS = ("absb_plan", "absb_step_form_used", "absb_status_offset", "absb_workspace_init", "absb_build_centroids", "absb_score", "absb_topk", "absb_sparse_decode",
           "absb_decode_fused", "absb_tail_init", "absb_append_token", "absb_head_recall", "absb_assign_block_sizes", "absb_stream_read",
           "absb_strerror", "absb_decode_fused_static")


class AbsbError(RuntimeError):
    def __init__(self, status: int, where: str):
        self.status = status
        super().__init__(f"{where}: {strerror(status)} (status {status})")


class _Layer(C.Structure):
    _fields_ = [("num_q_heads", C.c_int32), ("num_kv_heads", C.c_int32), ("head_dim", C.c_int32),
                ("page_size", C.c_int32), ("dtype", C.c_int32), ("block_repr", C.c_int32),
                ("block_size", C.c_void_p),
                ("kv_stride_page", C.c_int64), ("kv_stride_head", C.c_int64), ("kv_stride_tok", C.c_int64),
                ("sm_scale", C.c_float), ("sink_tokens", C.c_int32), ("recent_tokens", C.c_int32),
                ("selection", C.c_int32)]


class _Opts(C.Structure):
    _fields_ = [("step_form", C.c_int32), ("split_tokens", C.c_int32), ("score_chunk", C.c_int32),
                ("unit_tokens", C.c_int32), ("counters_zero", C.c_int32)]


class _Batch(C.Structure):
    _fields_ = [("batch", C.c_int32), ("pt_stride", C.c_int32),
                ("seq_lens_host", C.c_void_p), ("seq_lens", C.c_void_p),
                ("page_table", C.c_void_p), ("cent_off", C.c_void_p),
                ("budget_host", C.c_void_p), ("budget", C.c_void_p),
                ("cap_lens_host", C.c_void_p), ("qmin", C.c_void_p), ("opts", _Opts)]


_lib = None

# Argument types of the entry points: with them declared, integers, None, byref() records and c_void_p
# objects are converted by ctypes itself, so a call passes plain integers (addresses, sizes) and builds
# no wrapper objects.  P: an address or None.
_P, _REC = C.c_void_p, C.c_void_p
_ARGTYPES = {
    "absb_plan": [_REC, _REC, _P, _P, _P, _P],
    "absb_step_form_used": [_REC, _REC],
    "absb_status_offset": [_REC, _REC, _P],
    "absb_workspace_init": [_REC, _REC, _P, C.c_size_t, _P],
    "absb_build_centroids": [_REC, _REC, _P, _P, _P, _P, _P, C.c_size_t, _P],
    "absb_score": [_REC, _REC, _P, _P, _P, _P, _P, _P],
    "absb_topk": [_REC, _REC, _P, _P, _P, C.c_int32, _P, C.c_size_t, _P],
    "absb_sparse_decode": [_REC, _REC, _P, _P, _P, _P, _P, C.c_int32, _P, _P, _P, C.c_size_t, _P],
    "absb_decode_fused": [_REC, _REC, _P, _P, _P, _P, _P, _P, _P, _P, _P, _P, C.c_size_t, _P],
    "absb_decode_fused_static": [_REC, _REC, _P, _P, _P, _P, _P, _P, _P, _P, _P, _P],
    "absb_tail_init": [_REC, _REC, _P, _P, _P],
    "absb_append_token": [_REC, _REC, _P, _P, _P, _P, _P, _P, _P],
    "absb_head_recall": [_REC, _REC, _P, _P, _P, _P],
    "absb_stream_read": [_P, C.c_size_t, _P, _P],
}


def load() -> C.CDLL:
    """Load libabsb.so (built in-tree by paper_2605_12110_amd.build).  Raises if it is not there."""
    global _lib
    if _lib is None:
        if not os.path.exists(LIB_PATH):
            raise RuntimeError(f"{LIB_PATH} is missing: run `python -c 'import __graft_entry__ as g; g.build()'` "
                               "(there is no CPU fallback)")
        lib = C.CDLL(LIB_PATH)
        lib.absb_strerror.restype = C.c_char_p
        lib.absb_strerror.argtypes = [C.c_int]
        for name in EXPORTS:
            f = getattr(lib, name)            # fail loudly on a stale library
            if name in _ARGTYPES:
                f.argtypes = _ARGTYPES[name]
        _lib = lib
    return _lib


def strerror(status: int) -> str:
    return load().absb_strerror(int(status)).decode()


def _check(status: int, where: str) -> None:
    if status != OK:
        raise AbsbError(status, where)


def _ptr(t) -> Optional[int]:
    if t is None or isinstance(t, int):
        return t
    return t.data_ptr()


_raw_stream = None


def _stream(stream) -> int:
    """The raw hipStream_t: of a torch stream, an address, or (None) torch's current stream."""
    if stream is None:
        global _raw_stream
        if _raw_stream is None:
            import torch
            get, device = torch._C._cuda_getCurrentRawStream, torch.cuda.current_device
            device()                            # initialises the runtime, or raises where there is no GPU
            device = torch._C._cuda_getDevice
            _raw_stream = lambda: get(device())  # noqa: E731  (no Stream object per call)
        return _raw_stream()
    if isinstance(stream, int):
        return stream
    return stream.cuda_stream


_INT32 = np.dtype(np.int32)


def _i32_host(a: Optional[Sequence[int]]):
    """(contiguous int32 array to keep alive, its address); (None, None) for None."""
    if a is None:
        return None, None
    if type(a) is not np.ndarray or a.dtype != _INT32 or a.ndim != 1 or not a.flags.c_contiguous:
        a = np.ascontiguousarray(np.asarray(a), dtype=np.int32)
    try:
        return a, C.addressof(C.c_byte.from_buffer(a))
    except (TypeError, ValueError):             # a read-only or an empty array: the slower way
        return a, a.__array_interface__["data"][0]


@dataclass
class Layer:
    """Host description of a layer (mirrors absb_layer)."""
    num_q_heads: int
    num_kv_heads: int
    head_dim: int
    page_size: int
    dtype: int
    block_size: Sequence[int]
    kv_strides: Sequence[int]          # (page, head, token) in elements
    sm_scale: float = 0.0
    block_repr: int = REPR_MEAN
    sink_tokens: int = 0
    recent_tokens: int = 0
    selection: int = SELECT_GROUP

    def __setattr__(self, name, value):
        object.__setattr__(self, name, value)
        if not name.startswith("_"):
            object.__setattr__(self, "_c", None)       # any field change invalidates the cached C struct

    def c(self) -> _Layer:
        """The absb_layer record (built once per set of field values: marshalling stays off the hot path)."""
        if getattr(self, "_c", None) is None:
            self._bs, bs_p = _i32_host(self.block_size)
            sp, sh, st = (int(x) for x in self.kv_strides)
            self._c = _Layer(self.num_q_heads, self.num_kv_heads, self.head_dim, self.page_size, self.dtype,
                             int(self.block_repr),
                             bs_p, sp, sh, st, float(self.sm_scale), int(self.sink_tokens),
                             int(self.recent_tokens), int(self.selection))
        return self._c


@dataclass
class LaunchOpts:
    """How a call is enqueued (mirrors absb_launch_opts): all zero = the library's choices."""
    step_form: int = STEP_AUTO
    split_tokens: int = 0
    score_chunk: int = 0
    unit_tokens: int = 0
    counters_zero: int = 0


@dataclass
class Batch:
    """One decode step's batch (mirrors absb_batch).  Host arrays are numpy/sequences, device
    arrays are int32 torch tensors on the GPU (or None where an entry point does not need them)."""
    seq_lens_host: Sequence[int]
    budget_host: Optional[Sequence[int]] = None
    seq_lens: object = None
    page_table: object = None
    cent_off: object = None
    budget: object = None
    pt_stride: Optional[int] = None
    cap_lens_host: Optional[Sequence[int]] = None
    qmin: object = None
    opts: LaunchOpts = None

    def __post_init__(self):
        if self.opts is None:
            self.opts = LaunchOpts()

    def __setattr__(self, name, value):
        d = self.__dict__
        with _record_lock:
            d[name] = value
            if "_dirty" in d:
                d["_dirty"].add(name)

    def c(self) -> _Batch:
        """The absb_batch record.  Kept until a field is reassigned (a decode loop's lengths); then that field, and
        any other that was changed in place since, is carried over into a copy of the record, so a call in flight on
        another thread keeps the one it was given (with the host arrays it points into), and no thread gets
        a record from before a reassignment; the tensors must stay alive."""
        d = self.__dict__
        if d.get("_dirty", True):       # no record yet, or fields reassigned since (cleared only once the new one is in place)
            with _record_lock:
                self._renew(d)
        rec = d["_c"]
        o = self.opts                   # the options object may have been changed in place: looked at every time
        opts = (o.step_form, o.split_tokens, o.score_chunk, o.unit_tokens, o.counters_zero)
        if opts != rec._opts:
            rec.opts = _Opts(*(int(x) for x in opts))
            rec._opts = opts
        return rec

    def _renew(self, d) -> None:
        old = d.get("_c")
        rec = _Batch() if old is None else _Batch.from_buffer_copy(old)
        if old is None:
            rec._arrays, rec._at, rec._opts = {}, {}, None
            names = _BATCH_FIELDS
        else:
            rec._arrays, rec._at, rec._opts = dict(old._arrays), dict(old._at), old._opts
            names = set(d["_dirty"])
            # what is held by address only (tensors), or as a converted copy (lists), may have changed in place
            for name, arr in old._arrays.items():
                if d[name] is not arr:
                    names.add(name)
            for name, at in old._at.items():
                t = d[name]
                if (t if t is None or t.__class__ is int else t.data_ptr()) != at:
                    names.add(name)
            table = d["page_table"]
            if d["pt_stride"] is None and table is not None and table.shape[1] != rec.pt_stride:
                names.add("page_table")
        self._fill(rec, names)
        d["_c"] = rec
        d["_dirty"] = set()

    def _fill(self, rec, names) -> None:
        for name in names:
            value = getattr(self, name)
            if name in _BATCH_HOST_ARRAYS:
                rec._arrays[name], address = _i32_host(value)
                setattr(rec, name, address)
                if name == "seq_lens_host":
                    rec.batch = len(rec._arrays[name])
            elif name in _BATCH_TENSORS:
                rec._at[name] = address = _ptr(value)
                setattr(rec, name, address)
            if name in ("page_table", "pt_stride"):
                pts = self.pt_stride
                if pts is None:
                    pts = self.page_table.shape[1] if self.page_table is not None else 0
                rec.pt_stride = int(pts)


_record_lock = threading.RLock()    # of every batch: held for microseconds, and never around a call into the library
_BATCH_HOST_ARRAYS = frozenset(("seq_lens_host", "budget_host", "cap_lens_host"))
_BATCH_TENSORS = frozenset(("seq_lens", "page_table", "cent_off", "budget", "qmin"))
_BATCH_FIELDS = (*_BATCH_HOST_ARRAYS, *_BATCH_TENSORS, "pt_stride")


@dataclass
class PlanResult:
    cent_off: np.ndarray       # int32 [Bt*Hkv+1]
    total_centroids: int
    sel_stride: int
    workspace_bytes: int


def absb_plan(layer: Layer, batch: Batch) -> PlanResult:
    cl, cb = layer.c(), batch.c()
    nseg = cb.batch * layer.num_kv_heads
    off = np.zeros(max(nseg, 0) + 1, dtype=np.int32)
    total, stride, ws = C.c_int64(0), C.c_int32(0), C.c_size_t(0)
    _check(load().absb_plan(C.byref(cl), C.byref(cb), off.ctypes.data,
                            C.byref(total), C.byref(stride), C.byref(ws)), "absb_plan")
    return PlanResult(off, int(total.value), int(stride.value), int(ws.value))


def absb_build_centroids(layer: Layer, batch: Batch, k_cache, codes, qscale, qmin, workspace, stream=None) -> None:
    cl, cb = layer.c(), batch.c()
    _check(load().absb_build_centroids(C.byref(cl), C.byref(cb), _ptr(k_cache), _ptr(codes), _ptr(qscale),
                                       _ptr(qmin), _ptr(workspace), _nbytes(workspace),
                                       _stream(stream)), "absb_build_centroids")


def absb_score(layer: Layer, batch: Batch, q, codes, qscale, scores, score_exp=None, stream=None) -> None:
    cl, cb = layer.c(), batch.c()
    _check(load().absb_score(C.byref(cl), C.byref(cb), _ptr(q), _ptr(codes), _ptr(qscale), _ptr(scores),
                             _ptr(score_exp), _stream(stream)), "absb_score")


def absb_topk(layer: Layer, batch: Batch, scores, sel_idx, sel_cnt, sel_stride: int, workspace=None,
              stream=None) -> None:
    cl, cb = layer.c(), batch.c()
    _check(load().absb_topk(C.byref(cl), C.byref(cb), _ptr(scores), _ptr(sel_idx), _ptr(sel_cnt),
                            sel_stride, _ptr(workspace), _nbytes(workspace),
                            _stream(stream)), "absb_topk")


def absb_sparse_decode(layer: Layer, batch: Batch, q, k_cache, v_cache, sel_idx, sel_cnt, sel_stride: int,
                       out, lse, workspace, stream=None) -> None:
    cl, cb = layer.c(), batch.c()
    _check(load().absb_sparse_decode(C.byref(cl), C.byref(cb), _ptr(q), _ptr(k_cache), _ptr(v_cache),
                                     _ptr(sel_idx), _ptr(sel_cnt), sel_stride, _ptr(out), _ptr(lse),
                                     _ptr(workspace), _nbytes(workspace), _stream(stream)),
           "absb_sparse_decode")


def absb_decode_fused(layer: Layer, batch: Batch, q, codes, qscale, k_cache, v_cache, out, lse=None,
                      sel_idx_out=None, sel_cnt_out=None, workspace=None, stream=None) -> None:
    cl, cb = layer.c(), batch.c()
    _check(load().absb_decode_fused(C.byref(cl), C.byref(cb), _ptr(q), _ptr(codes), _ptr(qscale), _ptr(k_cache),
                                    _ptr(v_cache), _ptr(out), _ptr(lse), _ptr(sel_idx_out), _ptr(sel_cnt_out),
                                    _ptr(workspace), _nbytes(workspace), _stream(stream)),
           "absb_decode_fused")


def absb_decode_fused_static(layer: Layer, batch: Batch, q, codes, qscale, k_cache, v_cache, out, lse=None,
                             sel_idx_out=None, sel_cnt_out=None, stream=None) -> None:
    """The step on the library's built-in scratch array: no workspace argument, nothing allocated."""
    cl, cb = layer.c(), batch.c()
    _check(load().absb_decode_fused_static(C.byref(cl), C.byref(cb), _ptr(q), _ptr(codes), _ptr(qscale),
                                           _ptr(k_cache), _ptr(v_cache), _ptr(out), _ptr(lse), _ptr(sel_idx_out),
                                           _ptr(sel_cnt_out), _stream(stream)), "absb_decode_fused_static")


def absb_step_form_used(layer: Layer, batch: Batch) -> int:
    """The absb_step_form absb_decode_fused will use for this (layer, batch, batch.opts): 1, 2 or 3."""
    cl, cb = layer.c(), batch.c()
    n = load().absb_step_form_used(C.byref(cl), C.byref(cb))
    if n < 0:
        raise AbsbError(n, "absb_step_form_used")
    return int(n)


def absb_status_offset(layer: Layer, batch: Batch) -> int:
    cl, cb = layer.c(), batch.c()
    off = C.c_size_t(0)
    _check(load().absb_status_offset(C.byref(cl), C.byref(cb), C.byref(off)), "absb_status_offset")
    return int(off.value)


def absb_workspace_init(layer: Layer, batch: Batch, workspace, stream=None) -> None:
    cl, cb = layer.c(), batch.c()
    _check(load().absb_workspace_init(C.byref(cl), C.byref(cb), _ptr(workspace), _nbytes(workspace),
                                      _stream(stream)), "absb_workspace_init")


def absb_tail_init(layer: Layer, batch: Batch, k_cache, tail, stream=None) -> None:
    cl, cb = layer.c(), batch.c()
    _check(load().absb_tail_init(C.byref(cl), C.byref(cb), _ptr(k_cache), _ptr(tail), _stream(stream)),
           "absb_tail_init")


def absb_append_token(layer: Layer, batch: Batch, k_cache, codes, qscale, qmin, tail, clamped=None,
                      stream=None) -> None:
    cl, cb = layer.c(), batch.c()
    _check(load().absb_append_token(C.byref(cl), C.byref(cb), _ptr(k_cache), _ptr(codes), _ptr(qscale), _ptr(qmin),
                                    _ptr(tail), _ptr(clamped), _stream(stream)), "absb_append_token")


def absb_head_recall(layer: Layer, batch: Batch, lse_selected, lse_dense, recall, stream=None) -> None:
    cl, cb = layer.c(), batch.c()
    _check(load().absb_head_recall(C.byref(cl), C.byref(cb), _ptr(lse_selected), _ptr(lse_dense), _ptr(recall),
                                   _stream(stream)), "absb_head_recall")


def absb_assign_block_sizes(recall: np.ndarray, candidates: Sequence[int], tau: float):
    """recall [n_samples, n_heads, n_cand] f32 (host) -> (block size per head, mean recall [heads, cands])."""
    rec = np.ascontiguousarray(recall, dtype=np.float32)
    n, nh, nc = rec.shape
    cand = np.ascontiguousarray(candidates, dtype=np.int32)
    out = np.empty(nh, np.int32)
    mean = np.empty((nh, nc), np.float64)
    _check(load().absb_assign_block_sizes(C.c_int32(n), C.c_int32(nh), C.c_int32(nc),
                                          rec.ctypes.data_as(C.c_void_p), cand.ctypes.data_as(C.c_void_p),
                                          C.c_double(tau), out.ctypes.data_as(C.c_void_p),
                                          mean.ctypes.data_as(C.c_void_p)), "absb_assign_block_sizes")
    return out, mean


def absb_stream_read(src, sink, stream=None) -> None:
    _check(load().absb_stream_read(_ptr(src), _nbytes(src), _ptr(sink), _stream(stream)),
           "absb_stream_read")


def _nbytes(t) -> int:
    if t is None:
        return 0
    return t.numel() * t.element_size()
