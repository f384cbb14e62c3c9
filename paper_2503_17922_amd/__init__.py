"""Thin Python binding of libwkv (MI355X WindowKV window selection).

Argument marshalling only: every function below has the name and the arguments of the C entry
point it calls (see ``include/wkv.h``); tensors are handed over as raw device pointers and the
current torch stream as the HIP stream.  The calls made per layer or per token go through the compiled
module ``_native`` (``csrc/wkv_python.cpp``), the others through ctypes.  Nothing is computed here, and there is no fallback:
if the HIP library is missing, every call raises.
"""
from __future__ import annotations

import ctypes as C
import importlib
import os
from typing import List, Optional, Sequence

_HERE = os.path.dirname(os.path.abspath(__file__))
LIB_PATH = os.path.join(_HERE, "libwkv.so")

WKV_OK, WKV_ERR_INVALID_ARG, WKV_ERR_UNSUPPORTED, WKV_ERR_WORKSPACE, WKV_ERR_HIP = 0, -1, -2, -3, -4
WKV_F32, WKV_BF16, WKV_F16 = 0, 1, 2
WKV_KEEP_PADDING = 1          # Problem(flags=...): leave compact-cache rows past n_keep untouched
WKV_SCORE_TWO_PASS, WKV_SCORE_SINGLE_READ, WKV_DEBUG_WAIT_GIVES_UP = 2, 4, 8      # Problem(flags=...)
WKV_DECODE_KEEP_COUNT = 1     # DecodeShape(flags=...): n_valid is read but not advanced
WKV_MAX_BATCH, WKV_MAX_GROUPS, WKV_MAX_LAYERS, WKV_MAX_WIN = 64, 64, 64, 128
WKV_MAX_OBS_ROWS, WKV_MAX_WINDOWS = 256, 32768
WKV_N_STAGES = 4
STAGE_NAMES = ("score_stats", "score", "select", "gather")

EXPORTS = ("wkv_get_dims", "wkv_workspace_bytes", "wkv_get_workspace_layout", "wkv_score", "wkv_window_pool",
           "wkv_topk_windows", "wkv_gather_group", "wkv_compress_group", "wkv_compress_groups",
           "wkv_compress_groups_profiled", "wkv_group_budgets", "wkv_status_string", "wkv_last_error",
           "wkv_decode_workspace_bytes", "wkv_decode_step", "wkv_decode_step_static", "wkv_index_jaccard")
WKV_DECODE_STATIC_SCRATCH_BYTES = 8 << 20


class WkvError(RuntimeError):
    def __init__(self, status: int, message: str):
        super().__init__(f"wkv status {status}: {message}")
        self.status = status


class _Problem(C.Structure):
    _fields_ = [
        ("batch", C.c_int32), ("n_q_heads", C.c_int32), ("n_kv_heads", C.c_int32),
        ("head_dim", C.c_int32), ("w_obs", C.c_int32), ("max_seq_len", C.c_int32),
        ("dtype", C.c_int32), ("scale", C.c_float),
        ("seq_len", C.POINTER(C.c_int32)), ("win", C.POINTER(C.c_int32)),
        ("top_p", C.POINTER(C.c_int32)), ("k_windows", C.POINTER(C.c_int32)),
        ("q_stride_b", C.c_int64), ("q_stride_h", C.c_int64), ("q_stride_t", C.c_int64),
        ("kv_stride_b", C.c_int64), ("kv_stride_h", C.c_int64), ("kv_stride_t", C.c_int64),
        ("out_stride_b", C.c_int64), ("out_stride_h", C.c_int64), ("out_stride_t", C.c_int64),
        ("flags", C.c_int32),
    ]


class _DecodeShape(C.Structure):
    _fields_ = [("batch", C.c_int32), ("n_q_heads", C.c_int32), ("n_kv_heads", C.c_int32), ("head_dim", C.c_int32),
                ("dtype", C.c_int32), ("scale", C.c_float), ("capacity", C.c_int32),
                ("cache_stride_b", C.c_int64), ("cache_stride_h", C.c_int64), ("cache_stride_t", C.c_int64),
                ("flags", C.c_int32)]


class Dims(C.Structure):
    _fields_ = [("obs_rows", C.c_int32), ("t_stride", C.c_int32), ("nw_max", C.c_int32),
                ("k_max", C.c_int32), ("nkeep_max", C.c_int32), ("total_tokens", C.c_int64)]


class WorkspaceLayout(C.Structure):
    _fields_ = [("t_offset", C.c_size_t), ("s_offset", C.c_size_t), ("t_written", C.c_int32), ("s_written", C.c_int32)]


_lib = None
_calls = None


def native():
    """The compiled marshalling module.  Raises if it has not been built (there is no fallback)."""
    global _calls
    if _calls is None:
        lib()
        module = importlib.import_module("._native", __name__)
        module.bind(_current_stream, _structure, Problem, _Problem, DecodeShape, _DecodeShape)
        _calls = module
    return _calls


def _structure(o, kind):
    """The structure that a ctypes function with a pointer to ``kind`` as its first argument would get from ``o.ref()``."""
    r = o.ref()
    try:
        C.POINTER(kind).from_param(r)
    except TypeError as e:
        raise C.ArgumentError(f"argument 1: {e}") from None
    return r._obj if hasattr(r, "_obj") else r.contents        # of byref(), of a pointer


def _current_stream() -> int:
    import torch
    return torch.cuda.current_stream().cuda_stream


def lib() -> C.CDLL:
    """The loaded HIP library.  Raises if it has not been built (no CPU fallback exists)."""
    global _lib
    if _lib is not None:
        return _lib
    if not os.path.exists(LIB_PATH):
        raise RuntimeError(f"{LIB_PATH} is missing: build it with `python -m paper_2503_17922_amd.build` "
                           "(there is no fallback path)")
    l = C.CDLL(LIB_PATH)
    P, VP = C.POINTER(_Problem), C.c_void_p
    l.wkv_get_dims.argtypes = [P, C.POINTER(Dims)]; l.wkv_get_dims.restype = C.c_int
    l.wkv_workspace_bytes.argtypes = [P, C.c_int32]; l.wkv_workspace_bytes.restype = C.c_size_t
    l.wkv_get_workspace_layout.argtypes = [P, C.c_int32, C.POINTER(WorkspaceLayout)]
    l.wkv_get_workspace_layout.restype = C.c_int
    l.wkv_score.argtypes = [P, VP, VP, VP, VP, VP, C.c_size_t, VP]; l.wkv_score.restype = C.c_int
    l.wkv_window_pool.argtypes = [P, VP, VP, VP]; l.wkv_window_pool.restype = C.c_int
    l.wkv_topk_windows.argtypes = [P, VP, VP, VP, VP, VP]; l.wkv_topk_windows.restype = C.c_int
    l.wkv_gather_group.argtypes = [P, C.c_int32, C.POINTER(VP), C.POINTER(VP), VP, VP,
                                   C.POINTER(VP), C.POINTER(VP), VP]
    l.wkv_gather_group.restype = C.c_int
    l.wkv_compress_groups.argtypes = [P, C.c_int32, C.c_int32, C.POINTER(VP), C.POINTER(VP), C.POINTER(C.c_int32),
                                      C.POINTER(VP), C.POINTER(VP), C.POINTER(VP), C.POINTER(VP), VP, VP, VP, VP,
                                      C.c_size_t, VP]
    l.wkv_compress_groups.restype = C.c_int
    l.wkv_compress_group.argtypes = [P, C.c_int32, VP, VP, C.POINTER(VP), C.POINTER(VP), C.POINTER(VP), C.POINTER(VP),
                                     VP, VP, VP, VP, C.c_size_t, VP]
    l.wkv_compress_group.restype = C.c_int
    l.wkv_compress_groups_profiled.argtypes = l.wkv_compress_groups.argtypes + [C.POINTER(C.c_float)]
    l.wkv_compress_groups_profiled.restype = C.c_int
    l.wkv_group_budgets.argtypes = [C.c_double, C.c_int32, C.c_double, C.POINTER(C.c_double)]
    l.wkv_group_budgets.restype = C.c_int
    l.wkv_index_jaccard.argtypes = [P, C.c_int32, VP, VP, VP, VP]; l.wkv_index_jaccard.restype = C.c_int
    DP = C.POINTER(_DecodeShape)
    l.wkv_decode_workspace_bytes.argtypes = [DP]; l.wkv_decode_workspace_bytes.restype = C.c_size_t
    l.wkv_decode_step.argtypes = [DP, VP, VP, VP, VP, VP, VP, VP, VP, C.c_size_t, VP]; l.wkv_decode_step.restype = C.c_int
    l.wkv_decode_step_static.argtypes = [DP, VP, VP, VP, VP, VP, VP, VP, VP]; l.wkv_decode_step_static.restype = C.c_int
    l.wkv_status_string.argtypes = [C.c_int]; l.wkv_status_string.restype = C.c_char_p
    l.wkv_last_error.argtypes = []; l.wkv_last_error.restype = C.c_char_p
    _lib = l
    return l


def _check(status: int) -> None:
    if status != WKV_OK:
        l = lib()
        detail = l.wkv_last_error().decode() or l.wkv_status_string(status).decode()
        raise WkvError(status, detail)


def _i32(xs: Sequence[int]):
    return (C.c_int32 * len(xs))(*[int(x) for x in xs])


class Problem:
    """Host-side description of one batch (mirrors ``wkv_problem``).  Strides are in elements;
    ``None`` selects contiguous ``[B, H, T, d]`` tensors."""

    def __init__(self, *, n_q_heads: int, n_kv_heads: int, head_dim: int, w_obs: int,
                 seq_len: Sequence[int], win: Sequence[int], top_p: Sequence[int],
                 k_windows: Sequence[int], dtype: int, max_seq_len: Optional[int] = None,
                 scale: float = 0.0, q_strides=None, kv_strides=None, out_strides=None,
                 nkeep_max: Optional[int] = None, flags: int = 0):
        B = len(seq_len)
        self._keep = [_i32(seq_len), _i32(win), _i32(top_p), _i32(k_windows)]
        if max_seq_len is None:
            max_seq_len = max(seq_len) if B else 0
        d = head_dim
        q_strides = q_strides or (n_q_heads * w_obs * d, w_obs * d, d)
        kv_strides = kv_strides or (n_kv_heads * max_seq_len * d, max_seq_len * d, d)
        # contiguous compact caches have nkeep_max rows per head; that size is the library's to derive
        # (wkv_get_dims), so the strides start from a placeholder and are set once it is known
        self.c = _Problem(B, n_q_heads, n_kv_heads, head_dim, w_obs, max_seq_len, dtype, scale,
                          self._keep[0], self._keep[1], self._keep[2], self._keep[3],
                          *q_strides, *kv_strides, *(out_strides or (d, d, d)), flags)
        if out_strides is None:
            if nkeep_max is None:
                dims = Dims()
                if lib().wkv_get_dims(C.byref(self.c), C.byref(dims)) == WKV_OK:
                    nkeep_max = dims.nkeep_max
            if nkeep_max is not None:      # an invalid problem keeps the placeholder; every call rejects it anyway
                self.c.out_stride_b, self.c.out_stride_h, self.c.out_stride_t = n_kv_heads * nkeep_max * d, nkeep_max * d, d

    def ref(self):
        return C.byref(self.c)


def _ptr(t) -> C.c_void_p:
    return C.c_void_p(t.data_ptr()) if t is not None else C.c_void_p(0)


def _ptr_array(ts):
    return (C.c_void_p * len(ts))(*[t.data_ptr() if t is not None else 0 for t in ts])


def _stream(stream=None) -> C.c_void_p:
    if stream is None:
        stream = _current_stream()
    return C.c_void_p(int(stream))


def wkv_get_dims(problem: Problem) -> Dims:
    d = Dims()
    _check(lib().wkv_get_dims(problem.ref(), C.byref(d)))
    return d


def wkv_workspace_bytes(problem: Problem, n_groups: int = 1) -> int:
    n = lib().wkv_workspace_bytes(problem.ref(), n_groups)
    if n == 0:
        raise WkvError(WKV_ERR_INVALID_ARG, lib().wkv_last_error().decode())
    return int(n)


def wkv_get_workspace_layout(problem: Problem, n_groups: int = 1) -> WorkspaceLayout:
    lay = WorkspaceLayout()
    _check(lib().wkv_get_workspace_layout(problem.ref(), n_groups, C.byref(lay)))
    return lay


def wkv_score(problem, q_obs, k_first, lse_obs, t_out, workspace, stream=None) -> None:
    """``lse_obs``: float32 [batch, n_q_heads, w_obs] natural-log softmax normalisers, or None."""
    _check((_calls or native()).score(problem, q_obs, k_first, lse_obs, t_out, workspace, stream))


def wkv_window_pool(problem, t, s_out, stream=None) -> None:
    _check((_calls or native()).window_pool(problem, t, s_out, stream))


def wkv_topk_windows(problem, s, win_idx_out, tok_idx_out, n_keep_out, stream=None) -> None:
    _check((_calls or native()).topk_windows(problem, s, win_idx_out, tok_idx_out, n_keep_out, stream))


def wkv_gather_group(problem, k_layers, v_layers, tok_idx, n_keep, k_out_layers, v_out_layers,
                     stream=None) -> None:
    _check((_calls or native()).gather_group(problem, k_layers, v_layers, tok_idx, n_keep, k_out_layers, v_out_layers, stream))


class CompressCall:
    """``wkv_compress_groups`` with its host pointer arrays marshalled once, for callers that
    repeat the same call (the benchmark's timed loop)."""

    def __init__(self, problem, n_groups, gamma, q_obs_groups, lse_obs_groups, k_layers, v_layers, k_out_layers,
                 v_out_layers, win_idx_out, tok_idx_out, n_keep_out, workspace, k_windows_groups=None):
        self._keep = (problem, q_obs_groups, lse_obs_groups, k_layers, v_layers, k_out_layers, v_out_layers,
                      win_idx_out, tok_idx_out, n_keep_out, workspace)
        ws_bytes = workspace.numel() * workspace.element_size() if workspace is not None else 0
        lse_arr = _ptr_array(lse_obs_groups) if lse_obs_groups is not None else None
        kg_arr = None
        if k_windows_groups is not None:       # [n_groups][batch] nested sequence, row-major as the ABI wants
            kg_arr = _i32([k for row in k_windows_groups for k in row])
        self._args = (problem.ref(), n_groups, gamma, _ptr_array(q_obs_groups), lse_arr, kg_arr, _ptr_array(k_layers),
                      _ptr_array(v_layers), _ptr_array(k_out_layers), _ptr_array(v_out_layers),
                      _ptr(win_idx_out), _ptr(tok_idx_out), _ptr(n_keep_out), _ptr(workspace), ws_bytes)
        self._fn = lib().wkv_compress_groups
        self._fn_profiled = lib().wkv_compress_groups_profiled

    def __call__(self, stream=None) -> None:
        _check(self._fn(*self._args, _stream(stream)))

    def profiled(self, stream=None) -> List[float]:
        """``wkv_compress_groups_profiled``: the same call, returning per-kernel milliseconds."""
        ms = (C.c_float * WKV_N_STAGES)()
        _check(self._fn_profiled(*self._args, _stream(stream), ms))
        return list(ms)


def wkv_compress_groups(problem, n_groups, gamma, q_obs_groups, lse_obs_groups, k_layers, v_layers, k_out_layers,
                        v_out_layers, win_idx_out, tok_idx_out, n_keep_out, workspace, stream=None,
                        k_windows_groups=None) -> None:
    """The C entry point's ``k_windows_groups`` (between ``lse_obs_groups`` and ``k_layers`` there)
    is the trailing keyword here: a nested [n_groups][batch] sequence of ints, or None."""
    _check((_calls or native()).compress_groups(problem, n_groups, gamma, q_obs_groups, lse_obs_groups, k_windows_groups, k_layers,
                                                v_layers, k_out_layers, v_out_layers, win_idx_out, tok_idx_out, n_keep_out,
                                                workspace, stream))


def wkv_compress_group(problem, gamma, q_obs, lse_obs, k_layers, v_layers, k_out_layers, v_out_layers, win_idx_out,
                       tok_idx_out, n_keep_out, workspace, stream=None) -> None:
    _check((_calls or native()).compress_group(problem, gamma, q_obs, lse_obs, k_layers, v_layers, k_out_layers, v_out_layers,
                                                win_idx_out, tok_idx_out, n_keep_out, workspace, stream))


def wkv_index_jaccard(problem, n_sets, tok_idx, n_keep, jaccard_out, stream=None) -> None:
    _check(lib().wkv_index_jaccard(problem.ref(), n_sets, _ptr(tok_idx), _ptr(n_keep), _ptr(jaccard_out), _stream(stream)))


class DecodeShape:
    """Mirrors ``wkv_decode_shape``.  ``cache_strides`` in elements; ``None`` selects contiguous
    ``[B, Hkv, capacity, d]`` caches."""

    def __init__(self, *, batch: int, n_q_heads: int, n_kv_heads: int, head_dim: int, dtype: int, capacity: int,
                 scale: float = 0.0, cache_strides=None, flags: int = 0):
        cache_strides = cache_strides or (n_kv_heads * capacity * head_dim, capacity * head_dim, head_dim)
        self.c = _DecodeShape(batch, n_q_heads, n_kv_heads, head_dim, dtype, scale, capacity, *cache_strides, flags)

    def ref(self):
        return C.byref(self.c)


def wkv_decode_workspace_bytes(shape: DecodeShape) -> int:
    n = lib().wkv_decode_workspace_bytes(shape.ref())
    if n == 0:
        raise WkvError(WKV_ERR_INVALID_ARG, lib().wkv_last_error().decode())
    return int(n)


def wkv_decode_step(shape: DecodeShape, q_new, k_new, v_new, k_cache, v_cache, n_valid, out, workspace,
                    stream=None) -> None:
    _check((_calls or native()).decode_step(shape, q_new, k_new, v_new, k_cache, v_cache, n_valid, out, workspace, stream))


def wkv_decode_step_static(shape: DecodeShape, q_new, k_new, v_new, k_cache, v_cache, n_valid, out, stream=None) -> None:
    _check((_calls or native()).decode_step_static(shape, q_new, k_new, v_new, k_cache, v_cache, n_valid, out, stream))


def wkv_group_budgets(b_total: float, n_groups: int, lam: float) -> List[float]:
    out = (C.c_double * max(n_groups, 1))()
    _check(lib().wkv_group_budgets(b_total, n_groups, lam, out))
    return list(out)[:n_groups]

