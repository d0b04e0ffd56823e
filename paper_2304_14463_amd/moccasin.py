"""Python binding of libmoccasin_hip.so (C ABI in include/moccasin.h).

Argument marshalling only: every step of the evaluation runs in the HIP
kernels of the library.  Tensors are torch tensors on the GPU (torch is used
for device memory and streams); graph arrays are host numpy arrays.  There is
no CPU fallback: a missing library or GPU raises.
"""
from __future__ import annotations

import ctypes
import os

import numpy as np

_PKG = os.path.dirname(os.path.abspath(__file__))
LIB_PATH = os.path.join(_PKG, "libmoccasin_hip.so")
_lib = None
_torch = None
_native = None

MOC_MAX_T = 19455
MOC_ABI_VERSION = 2

# numpy views of the result structs of include/moccasin.h
RESULT_DTYPE = np.dtype([("peak", "<i8"), ("duration", "<i8"), ("violations", "<i4"), ("feasible", "<i4")])
MOVE_SCORE_DTYPE = np.dtype([("violations", "<i4"), ("peak", "<i4")])
BEST_MOVE_DTYPE = np.dtype([("move", "<i4"), ("violations", "<i4"), ("peak", "<i8")])
TOGGLE_SCORE_DTYPE = np.dtype([("violations", "<i4"), ("peak", "<i4"), ("duration", "<i8")])
DECODE_RESULT_DTYPE = np.dtype([("status", "<i4"), ("length", "<i4"), ("peak", "<i8"), ("duration", "<i8")])

EXPORTS = ("moc_graph_upload", "moc_graph_info", "moc_eval_batch", "moc_eval_batch_noalloc", "moc_graph_set_order", "moc_eval_batch_staged", "moc_eval_neighbours", "moc_eval_toggles",
           "moc_eval_cuts", "moc_eval_cuts_keep", "moc_search_cuts", "moc_search_two_phase", "moc_search_moves", "moc_decode_batch", "moc_graph_free", "moc_abi_version", "moc_strerror", "moc_last_hip_error")


class MoccasinError(RuntimeError):
    def __init__(self, code, where):
        self.code = code
        msg = lib().moc_strerror(code).decode()
        hip = lib().moc_last_hip_error() if code == -4 else 0
        super().__init__(f"{where}: {msg} (code {code}" + (f", hipError {hip})" if hip else ")"))


def lib():
    """Load the shared library (build it first with `python -m paper_2304_14463_amd.build`)."""
    global _lib
    if _lib is None:
        if not os.path.exists(LIB_PATH):
            raise FileNotFoundError(f"{LIB_PATH} is not built; run python -m paper_2304_14463_amd.build")
        L = ctypes.CDLL(LIB_PATH)
        # A library of another version may write where this binding gives it no room
        # (moc_search_two_phase's workspaces): it is refused before any call.
        version = L.moc_abi_version() if hasattr(L, "moc_abi_version") else 1
        if version != MOC_ABI_VERSION:
            raise RuntimeError(f"{LIB_PATH} has interface version {version}, this binding needs {MOC_ABI_VERSION}; "
                               "run python -m paper_2304_14463_amd.build")
        P, I32, I64, VP = ctypes.POINTER, ctypes.c_int32, ctypes.c_int64, ctypes.c_void_p
        L.moc_graph_upload.argtypes = [I32, VP, VP, VP, VP, I64, I32, P(VP)]
        L.moc_graph_upload.restype = ctypes.c_int
        L.moc_graph_info.argtypes = [VP, P(I32), P(I32), P(I32), P(I32)]
        L.moc_graph_info.restype = ctypes.c_int
        L.moc_eval_batch.argtypes = [VP, I64, VP, VP, VP, VP, VP]
        L.moc_eval_batch.restype = ctypes.c_int
        L.moc_eval_batch_noalloc.argtypes = [VP, I64, VP, VP, VP, VP, VP]
        L.moc_eval_batch_noalloc.restype = ctypes.c_int
        L.moc_graph_set_order.argtypes = [VP, VP]
        L.moc_graph_set_order.restype = ctypes.c_int
        L.moc_eval_batch_staged.argtypes = [VP, I64, VP, VP, VP, VP, VP]
        L.moc_eval_batch_staged.restype = ctypes.c_int
        L.moc_eval_neighbours.argtypes = [VP, I64, VP, VP, VP, I32, VP, VP, VP]
        L.moc_eval_neighbours.restype = ctypes.c_int
        L.moc_eval_toggles.argtypes = [VP, I64, VP, VP, VP, VP, VP]
        L.moc_eval_toggles.restype = ctypes.c_int
        L.moc_eval_cuts.argtypes = [VP, I64, VP, VP, VP, VP, VP, VP]
        L.moc_eval_cuts.restype = ctypes.c_int
        L.moc_eval_cuts_keep.argtypes = [VP, I64, VP, VP, VP, VP, VP, VP]
        L.moc_eval_cuts_keep.restype = ctypes.c_int
        L.moc_search_two_phase.argtypes = [VP, I64, VP, VP, VP, I32, I32, I32, VP, VP, VP, VP, VP, VP, VP, VP, VP]
        L.moc_search_two_phase.restype = ctypes.c_int
        L.moc_search_cuts.argtypes = [VP, I64, VP, VP, VP, I32, VP, VP, VP]
        L.moc_search_cuts.restype = ctypes.c_int
        L.moc_search_moves.argtypes = [VP, I64, VP, VP, VP, I32, I32, VP, VP, VP, VP]
        L.moc_search_moves.restype = ctypes.c_int
        L.moc_decode_batch.argtypes = [VP, I64, VP, VP, VP, VP, VP]
        L.moc_decode_batch.restype = ctypes.c_int
        L.moc_graph_free.argtypes = [VP]
        L.moc_graph_free.restype = None
        L.moc_strerror.argtypes = [ctypes.c_int]
        L.moc_strerror.restype = ctypes.c_char_p
        L.moc_last_hip_error.argtypes = []
        L.moc_last_hip_error.restype = ctypes.c_int
        # the calls that _candidates.evaluate makes itself
        L.address = {name: ctypes.cast(getattr(L, name), VP).value for name in ("moc_eval_batch", "moc_eval_batch_staged", "moc_eval_toggles")}
        _lib = L
    return _lib


def _check(code, where):
    if code != 0:
        raise MoccasinError(code, where)


def _host(arr, n):
    a = np.ascontiguousarray(arr, dtype=np.int32).reshape(-1)
    if a.shape[0] != n:
        raise ValueError(f"expected {n} int32 values, got {a.shape[0]}")
    return a


def _tc():
    """torch, imported on first use (device memory and streams)."""
    global _torch
    if _torch is None:
        import torch
        _torch = torch
    return _torch


def _stream_handle(stream):
    # The raw handle of the current device's current stream, without a Stream object in between:
    # small calls are bound by what happens on the host before their launch.
    if stream is None:
        torch = _tc()
        return torch._C._cuda_getCurrentRawStream(torch.cuda.current_device())
    return stream.cuda_stream


def _on(stream):
    """Context in which tensors are allocated for use on `stream`: a workspace that this module
    allocates and drops while kernels queued on `stream` still use it must belong to that
    stream for torch's allocator, or it could be handed to work on another stream too early."""
    import contextlib
    return _tc().cuda.stream(stream) if stream is not None else contextlib.nullcontext()


class Graph:
    """Handle of an uploaded problem instance (moc_graph_upload / moc_graph_free)."""

    def __init__(self, handle, n, m, C):
        self._h = handle
        self.n, self.m, self.C, self.T = n, m, C, n * C

    def free(self):
        if self._h is not None:
            lib().moc_graph_free(self._h)
            self._h = None

    def __del__(self):
        try:
            self.free()
        except Exception:
            pass


def moc_graph_upload(n, in_ptr, in_idx, size, dur, budget, C) -> Graph:
    in_ptr = _host(in_ptr, n + 1)
    m = int(in_ptr[-1])
    in_idx = _host(in_idx, len(np.asarray(in_idx).reshape(-1)))
    size, dur = _host(size, n), _host(dur, n)
    h = ctypes.c_void_p()
    code = lib().moc_graph_upload(n, in_ptr.ctypes.data, in_idx.ctypes.data if in_idx.size else None,
                                  size.ctypes.data, dur.ctypes.data, int(budget), int(C), ctypes.byref(h))
    _check(code, "moc_graph_upload")
    return Graph(h, n, m, int(C))


def _candidates():
    """The native part of the binding (binding/candidates.cpp), loaded on first use: it needs torch."""
    global _native
    if _native is None:
        _tc()
        try:
            from . import _candidates as native   # built with the library
        except ImportError as err:
            raise RuntimeError(f"{_PKG}: the binding's native part does not load ({err}); run python -m paper_2304_14463_amd.build") from err
        if getattr(native, "abi_version", None) != MOC_ABI_VERSION:
            raise RuntimeError(f"{native.__file__}: ABI version {getattr(native, 'abi_version', None)}, expected {MOC_ABI_VERSION}; "
                               "run python -m paper_2304_14463_amd.build")
        _native = native
    return _native


def _cand_ptrs(g, starts, ends, active):
    """(B, addresses of the three arrays)"""
    return (_native or _candidates()).pointers(g.T, starts, ends, active)


def _room(out, wanted, like, size, *dims):
    """(tensor, address) of a result: the caller's, or a new one if it is wanted, or (None, None)"""
    if out is not None:
        return out, out.data_ptr()
    return _candidates().empty(like, size, *dims) if wanted else (None, None)


def _evaluate(name, g, starts, ends, active, out, per, size, stream):
    code, out = (_native or _candidates()).evaluate((_lib or lib()).address[name], g._h.value if g._h is not None else None, g.T,
                                                    starts, ends, active, out, per, size, _stream_handle(stream))
    if code != 0:
        raise MoccasinError(code, name)
    return out


def moc_eval_batch(g: Graph, starts, ends, active, out=None, stream=None):
    """Evaluate B candidates; returns a uint8 CUDA tensor [B][24] holding moc_result records
    (see results_to_numpy).  Asynchronous on `stream` (default: torch's current stream)."""
    return _evaluate("moc_eval_batch", g, starts, ends, active, out, 0, RESULT_DTYPE.itemsize, stream)


def moc_eval_batch_noalloc(g: Graph, starts, ends, active, out, stream=None):
    """moc_eval_batch with the work counters in the library's static device array; `out` is the
    caller's uint8 CUDA tensor [B][24].  Nothing is allocated, here or in the library."""
    B, ps, pe, pa = _cand_ptrs(g, starts, ends, active)
    if not (out.is_cuda and out.is_contiguous() and out.numel() * out.element_size() >= B * RESULT_DTYPE.itemsize):
        raise ValueError("out must be a contiguous CUDA tensor of at least B * 24 bytes")
    code = lib().moc_eval_batch_noalloc(g._h, B, ps, pe, pa, out.data_ptr(), _stream_handle(stream))
    _check(code, "moc_eval_batch_noalloc")
    return out


def moc_graph_set_order(g: Graph, order):
    """Give the graph the topological order of the stage-restricted domain (host array [n])."""
    order = _host(order, g.n)
    _check(lib().moc_graph_set_order(g._h, order.ctypes.data), "moc_graph_set_order")


def moc_eval_batch_staged(g: Graph, starts, ends, active, out=None, stream=None):
    """Evaluate B candidates in the stage-restricted domain; returns a uint8 CUDA tensor [B][24]
    of moc_result records."""
    return _evaluate("moc_eval_batch_staged", g, starts, ends, active, out, 0, RESULT_DTYPE.itemsize, stream)


def moc_eval_neighbours(g: Graph, starts, ends, active, R, want_moves=True, want_best=True, out_moves=None,
                        out_best=None, stream=None):
    """Score all single-field moves of B candidates.  Returns (moves, best): uint8 CUDA tensors
    [B][T*4R][8] (moc_move_score) and [B][16] (moc_best_move), or None where not requested."""
    B, ps, pe, pa = _cand_ptrs(g, starts, ends, active)
    out_moves, pm = _room(out_moves, want_moves, starts, 1, B, g.T * 4 * R, MOVE_SCORE_DTYPE.itemsize)
    out_best, pb = _room(out_best, want_best, starts, 1, B, BEST_MOVE_DTYPE.itemsize)
    code = lib().moc_eval_neighbours(g._h, B, ps, pe, pa, int(R), pm, pb, _stream_handle(stream))
    _check(code, "moc_eval_neighbours")
    return out_moves, out_best


def moc_eval_toggles(g: Graph, starts, ends, active, out=None, stream=None):
    """Score the B x T candidates that differ from a base in one active flag.  Returns a uint8
    CUDA tensor [B][T][16] (moc_toggle_score)."""
    return _evaluate("moc_eval_toggles", g, starts, ends, active, out, g.T, TOGGLE_SCORE_DTYPE.itemsize, stream)


def moc_eval_cuts(g: Graph, starts, ends, active, want_moves=True, want_best=False, out_moves=None, out_best=None,
                  stream=None, keep_inputs=False):
    """Score the B x m*C cut-and-recompute moves.  Returns (uint8 CUDA tensor [B][m*C][16] of
    moc_cut_score or None, uint8 CUDA tensor [B][16] of moc_best_move or None)."""
    B, ps, pe, pa = _cand_ptrs(g, starts, ends, active)
    out_moves, pm = _room(out_moves, want_moves, starts, 1, B, g.m * g.C, TOGGLE_SCORE_DTYPE.itemsize)
    out_best, pb = _room(out_best, want_best, starts, 1, B, BEST_MOVE_DTYPE.itemsize)
    call = lib().moc_eval_cuts_keep if keep_inputs else lib().moc_eval_cuts
    code = call(g._h, B, ps, pe, pa, pm, pb, _stream_handle(stream))
    _check(code, "moc_eval_cuts")
    return out_moves, out_best


def moc_search_cuts(g: Graph, starts, ends, active, max_steps, work_best=None, out_steps=None, stream=None):
    """Greedy descent by cut-and-recompute moves, in place.  Returns the int32 CUDA tensor [B] of
    moves applied per candidate."""
    torch = _tc()
    B, ps, pe, pa = _cand_ptrs(g, starts, ends, active)
    with _on(stream):
        if work_best is None:
            work_best = torch.empty((B, BEST_MOVE_DTYPE.itemsize), dtype=torch.uint8, device=starts.device)
        if out_steps is None:
            out_steps = torch.empty((B,), dtype=torch.int32, device=starts.device)
    code = lib().moc_search_cuts(g._h, B, ps, pe, pa, int(max_steps), work_best.data_ptr(),
                                 out_steps.data_ptr(), _stream_handle(stream))
    _check(code, "moc_search_cuts")
    return out_steps


def moc_search_two_phase(g: Graph, starts, ends, active, max_cuts, max_merges, K=64, stream=None):
    """Two-phase local search in place (cuts that keep the inputs towards the budget, then merges
    that lower the duration).  Returns (cuts, merges): int32 CUDA tensors [B] of moves applied."""
    torch = _tc()
    B, ps, pe, pa = _cand_ptrs(g, starts, ends, active)
    if B > 0 and max_merges > 0 and not 1 <= K <= 0x7FFFFFFF // B:   # the call's limit, before K becomes an int32
        raise MoccasinError(-1, "moc_search_two_phase")
    dev = starts.device
    with _on(stream):
        work_best = torch.empty((B, BEST_MOVE_DTYPE.itemsize), dtype=torch.uint8, device=dev)
        cuts = torch.empty((B,), dtype=torch.int32, device=dev)
        merges = torch.empty((B,), dtype=torch.int32, device=dev)
    P = lambda t: t.data_ptr() if t.numel() else None
    unused = P(work_best)   # the call asks for the second phase's workspaces and does not use them
    code = lib().moc_search_two_phase(g._h, B, ps, pe, pa, int(max_cuts), int(max_merges), int(K), P(work_best), unused,
                                      unused, unused, unused, unused, P(cuts), P(merges), _stream_handle(stream))
    _check(code, "moc_search_two_phase")
    return cuts, merges


def moc_search_moves(g: Graph, starts, ends, active, R, max_steps, out_steps=None, stream=None):
    """Greedy descent by single-field start/end moves of radius R, in place.  Returns the int32
    CUDA tensor [B] of moves applied per candidate."""
    torch = _tc()
    B, ps, pe, pa = _cand_ptrs(g, starts, ends, active)
    with _on(stream):
        work_best = torch.empty((B, BEST_MOVE_DTYPE.itemsize), dtype=torch.uint8, device=starts.device)
        if out_steps is None:
            out_steps = torch.empty((B,), dtype=torch.int32, device=starts.device)
    unused = work_best.data_ptr()   # the call asks for work_results and does not use them
    code = lib().moc_search_moves(g._h, B, ps, pe, pa, int(R), int(max_steps), unused, work_best.data_ptr(),
                                  out_steps.data_ptr(), _stream_handle(stream))
    _check(code, "moc_search_moves")
    return out_steps


def moc_decode_batch(g: Graph, starts, active, want_seq=True, out=None, out_seq=None, stream=None):
    """Decode B candidates to their sequences.  Returns (uint8 CUDA tensor [B][24] of
    moc_decode_result, int32 CUDA tensor [B][T] of sequences or None)."""
    B, ps, _, pa = _cand_ptrs(g, starts, None, active)
    out, po = _room(out, True, starts, 1, B, DECODE_RESULT_DTYPE.itemsize)
    out_seq, pq = _room(out_seq, want_seq, starts, 4, B, g.T)
    code = lib().moc_decode_batch(g._h, B, ps, pa, po, pq, _stream_handle(stream))
    _check(code, "moc_decode_batch")
    return out, out_seq


def results_to_numpy(out, dtype=RESULT_DTYPE):
    """Copy a record tensor to the host (synchronises) and view it as a structured array."""
    host = out.cpu().numpy()
    return host.reshape(-1).view(dtype).reshape(host.shape[:-1])
