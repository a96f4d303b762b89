"""Python binding of libLouisKV.

Each function passes torch tensors to the C ABI of include/louiskv.h (pointers,
sizes, the current HIP stream; marshalled natively, csrc/binding.cpp) and
raises LouisKVError on a non-zero status.  All arithmetic happens in the library's HIP kernels; if the
library is not built this module fails loudly instead of computing anything.
"""
from __future__ import annotations

import ctypes
import os
from typing import Optional, Sequence

import torch

_HERE = os.path.dirname(os.path.abspath(__file__))
LIB_PATH = os.path.join(_HERE, "liblouiskv.so")

F32, BF16 = 0, 1
REF_PREV, REF_ANCHOR = 0, 1

_P = ctypes.c_void_p
_I32 = ctypes.c_int32
_I64 = ctypes.c_int64
_SZ = ctypes.c_size_t
_F = ctypes.c_float
_D = ctypes.c_double

_SIGS = {
    "louiskv_abi_version": (ctypes.c_int, []),
    "louiskv_status_str": (ctypes.c_char_p, [ctypes.c_int]),
    "louiskv_last_error": (ctypes.c_char_p, []),
    "louiskv_window_info": (ctypes.c_int, [_I32, _I32, _I32, _P, _P, _P, _P]),
    "louiskv_cluster_prefill_workspace_size": (_SZ, [_I64, _I32, _I32, _I32, _I32]),
    "louiskv_cluster_prefill": (ctypes.c_int, [
        _P, _I32, _I64, _I32, _I32, _I32, _I32, _P,
        _P, _I32, _P, _P, _P, _P,
        _P, _P, _P, _I64, _I32, _P, _P, _SZ, _P]),
    "louiskv_pack_pool": (ctypes.c_int, [_P, _P, _I32, _I64, _I32, _I32, _P, _P, _P, _I64, _I32, _P]),
    "louiskv_cluster_prefill_pipelined_workspace_size": (_SZ, [_I64, _I32, _I32, _I32, _I32, _I32, _I32]),
    "louiskv_cluster_prefill_pipelined": (ctypes.c_int, [
        _P, _I32, _I64, _I32, _I32, _I32, _I32, _P,
        _P, _I32, _P, _P, _P, _P,
        _P, _P, _P, _I64, _I32, _I64, _I32, _P, _I64, _P, _SZ, _P, _P]),
    "louiskv_kmeans_assign": (ctypes.c_int, [_P, _I32, _I64, _I32, _I32, _I32, _P, _I32, _P, _P, _SZ, _P]),
    "louiskv_kmeans_update": (ctypes.c_int, [_P, _I32, _I64, _I32, _I32, _I32, _P, _P, _P, _I32, _P, _P, _SZ, _P]),
    "louiskv_segment_output": (ctypes.c_int, [
        _P, _P, _I32, _I64, _I32, _P, _P, _I32, _I32, _I32,
        _P, _P, _P, _I32, _I32, _P, _P, _I64, _I32, _I32, _P]),
    "louiskv_boundary_check": (ctypes.c_int, [_P, _P, _I32, _I64, _I32, _I32, _D, _I32, _I32, _P, _P, _P]),
    "louiskv_retrieve_workspace_size": (_SZ, [_I64, _I32, _I32]),
    "louiskv_retrieve": (ctypes.c_int, [
        _P, _I32, _I64, _I32, _I32, _I32, _D,
        _P, _P, _P, _I32, _I32,
        _P, _P, _I64, _I32, _I32, _P,
        _P, _P, _P, _P, _P, _P, _P, _SZ, _P]),
    "louiskv_retrieve_rows_workspace_size": (_SZ, [_I64, _I32]),
    "louiskv_retrieve_rows": (ctypes.c_int, [
        _P, _I32, _I64, _I32, _I32, _I32, _D,
        _P, _P, _P, _I32, _I32, _I32, _P,
        _P, _P, _P, _P, _P, _P, _SZ, _P]),
    "louiskv_sparse_decode_attn_rows_workspace_size": (_SZ, [_I64, _I32, _I32, _I32, _I32]),
    "louiskv_sparse_decode_attn_rows": (ctypes.c_int, [
        _P, _I32, _I64, _I32, _I32, _I32, _F,
        _P, _P, _I64, _P, _P, _I32, _P, _P, _I32, _I32, _I32,
        _P, _I32, _P, _P, _SZ, _P]),
    "louiskv_decode_step_workspace_size": (_SZ, [_I64, _I32, _I32, _I32, _I32, _I32]),
    "louiskv_decode_step_cached_workspace_size": (_SZ, [_I64, _I32, _I32, _I32, _I32, _I32]),
    "louiskv_decode_step": (ctypes.c_int, [
        _P, _P, _I32, _I64, _I32, _I32, _I32, _D, _I32, _I32, _P, _P,
        _P, _P, _P, _P, _I32, _I32, _P, _P, _P, _I32, _I32,
        _P, _P, _I64, _I32, _I32, _P, _P, _P, _P, _P, _P, _I32, _P, _P, _SZ, _P]),
    "louiskv_decode_step_cached": (ctypes.c_int, [
        _P, _P, _I32, _I64, _I32, _I32, _I32, _D, _I32, _I32, _P, _P,
        _P, _P, _P, _P, _I32, _I32, _P, _P, _P, _I32, _I32,
        _P, _P, _I64, _I32, _I32, _I32, _I32, _P, _P, _P, _P, _P, _P,
        _P, _P, _P, _P, _P, _P, _I32, _P, _P, _SZ, _P]),
    "louiskv_sparse_decode_attn_rows_noalloc": (ctypes.c_int, [
        _P, _I32, _I64, _I32, _I32, _I32, _F,
        _P, _P, _I64, _P, _P, _I32, _P, _P, _I32, _I32, _I32,
        _P, _I32, _P, _P]),
    "louiskv_fire_every": (ctypes.c_int, [_P, _I64, _I32, _I32, _P]),
    "louiskv_decode_prologue": (ctypes.c_int, [
        _P, _P, _I32, _I64, _I32, _I32, _D, _I32, _I32, _P, _P,
        _P, _P, _I64, _P, _P, _I32, _I32, _I32, _P, _P, _P, _I32, _I32, _P, _P, _I64, _I32, _I32, _P]),
    "louiskv_page_prefill": (ctypes.c_int, [
        _P, _P, _I32, _I64, _I32, _I32, _I32, _P, _I32, _P, _P, _P, _P, _I64, _I32, _P]),
    "louiskv_retrieve_rows_per_head": (ctypes.c_int, [
        _P, _I32, _I64, _I32, _I32, _I32, _D,
        _P, _P, _P, _I32, _I32, _I32, _P,
        _P, _P, _P, _P, _P, _P, _SZ, _P]),
    "louiskv_sparse_decode_attn_rows_per_head": (ctypes.c_int, [
        _P, _I32, _I64, _I32, _I32, _I32, _F,
        _P, _P, _I64, _P, _P, _I32, _P, _P, _I32, _I32, _I32,
        _P, _I32, _P, _P, _SZ, _P]),
    "louiskv_sparse_decode_attn_workspace_size": (_SZ, [_I64, _I32, _I32, _I32, _I32]),
    "louiskv_sparse_decode_attn": (ctypes.c_int, [
        _P, _I32, _I64, _I32, _I32, _I32, _F,
        _P, _P, _P, _I32, _P, _P, _I32, _I32, _I32,
        _P, _I32, _P, _P, _SZ, _P]),
    "louiskv_segment_state_ints": (_SZ, [_I32]),
    "louiskv_segment_state_init": (ctypes.c_int, [_P, _I64, _I32, _I32, _P]),
    "louiskv_segment_output_boundary": (ctypes.c_int, [
        _P, _P, _I32, _I64, _I32, _I32, _P, _P, _I32, _I32, _I32, _P, _P,
        _P, _P, _P, _I32, _I32, _P, _P, _I64, _I32, _I32, _P]),
    "louiskv_retrieve_seg": (ctypes.c_int, [
        _P, _I32, _I64, _I32, _I32, _I32, _D,
        _P, _P, _P, _I32, _I32, _P, _I32,
        _P, _P, _I64, _I32, _I32, _P,
        _P, _P, _P, _P, _P, _P, _P, _SZ, _P]),
    "louiskv_retrieve_rows_seg": (ctypes.c_int, [
        _P, _I32, _I64, _I32, _I32, _I32, _D,
        _P, _P, _P, _I32, _I32, _P, _I32, _I32, _P,
        _P, _P, _P, _P, _P, _P, _SZ, _P]),
    "louiskv_sparse_decode_attn_seg": (ctypes.c_int, [
        _P, _I32, _I64, _I32, _I32, _I32, _F,
        _P, _P, _P, _I32, _P, _P, _I32, _P, _I32,
        _P, _I32, _P, _P, _SZ, _P]),
    "louiskv_sparse_decode_attn_rows_seg": (ctypes.c_int, [
        _P, _I32, _I64, _I32, _I32, _I32, _F,
        _P, _P, _I64, _P, _P, _I32, _P, _P, _I32, _P, _I32,
        _P, _I32, _P, _P, _SZ, _P]),
    "louiskv_retrieve_delta_workspace_size": (_SZ, [_I64, _I32, _I32]),
    "louiskv_retrieve_delta": (ctypes.c_int, [
        _P, _I32, _I64, _I32, _I32, _I32, _D,
        _P, _P, _P, _I32, _I32, _P, _I32,
        _P, _P, _I64, _I32, _I32, _P,
        _P, _P, _P, _P, _P, _P, _P, _P, _P, _P, _SZ, _P]),
    "louiskv_retrieve_cached": (ctypes.c_int, [
        _P, _I32, _I64, _I32, _I32, _I32, _D,
        _P, _P, _P, _I32, _I32, _P, _I32,
        _P, _P, _I64, _I32, _I32, _I32, _I32, _P,
        _P, _P, _P, _P, _P, _P, _P, _P, _P, _P, _P, _SZ, _P]),
}

EXPORTED = sorted(_SIGS)

_lib = None


class LouisKVError(RuntimeError):
    def __init__(self, status: int, message: str):
        super().__init__(f"libLouisKV status {status}: {message}")
        self.status = status


def load_library(path: Optional[str] = None) -> ctypes.CDLL:
    """The library for ctypes callers of its C ABI (loaded once; another build's
    by path); raises if it has not been built.  The functions of this module
    do not call through it: _native() does, into the in-tree library."""
    global _lib
    if _lib is not None and path is None:
        return _lib
    p = path or LIB_PATH
    if not os.path.exists(p):
        raise RuntimeError(f"libLouisKV is not built ({p} missing); run `python -m paper_2510_11292_amd.build`")
    lib = ctypes.CDLL(p)
    for name, (res, args) in _SIGS.items():
        fn = getattr(lib, name)
        fn.restype = res
        fn.argtypes = args
    if path is None:
        _lib = lib
    return lib


_binding = None


def _native():
    """The native marshalling of the ABI calls (csrc/binding.cpp)."""
    global _binding
    if _binding is None:
        if not os.path.exists(LIB_PATH):
            load_library()   # raises
        try:
            from . import _binding as m
        except ImportError as e:
            raise RuntimeError(f"the binding of libLouisKV is not built ({e}); "
                               f"run `python -m paper_2510_11292_amd.build`") from e
        _binding = m
    return _binding


def _check(status: int) -> None:
    if status != 0:
        raise LouisKVError(status, _native().last_error())   # the text of the library that ran the call


def _dtype_code(t: torch.Tensor) -> int:
    if t.dtype == torch.float32:
        return F32
    if t.dtype == torch.bfloat16:
        return BF16
    raise TypeError(f"unsupported dtype {t.dtype}")


def _ws(workspace: Optional[torch.Tensor], device, size, *args):
    """The workspace and its bytes; one of size(*args) bytes where none is given."""
    if workspace is None:
        workspace = torch.empty(max(int(size(*args)), 1), dtype=torch.uint8, device=device)
        return workspace, workspace.numel()
    return workspace, workspace.nbytes


def abi_version() -> int:
    return _native().abi_version()


def window_info(step: int, window: int, seg_len: int):
    """(evicted_segment or -1, n_evicted, n_local, local_start) after storing token `step`."""
    out = _native().window_info(step, window, seg_len)
    if type(out) is int:
        _check(out)
    return out


def cluster_prefill_workspace_size(n_slices, n_tokens, n_clusters, dtype_code, d=128) -> int:
    return _native().cluster_prefill_workspace_size(n_slices, n_tokens, d, n_clusters, dtype_code)


def cluster_prefill(keys, n_clusters: int, n_iters: int, init_idx, reps, unit_start, unit_size, assign, perm,
                    values=None, k_pool=None, v_pool=None, pool_on_host: bool = False,
                    iter_events: Optional[Sequence] = None, workspace=None, stream=None):
    s, n, d = keys.shape
    dt = _dtype_code(keys)
    ws, wsb = _ws(workspace, keys.device, cluster_prefill_workspace_size, s, n, n_clusters, dt, d)
    pool_rows = k_pool.shape[1] if k_pool is not None else (v_pool.shape[1] if v_pool is not None else 0)
    ev = None
    if iter_events is not None:
        arr = (ctypes.c_void_p * len(iter_events))(*[e.cuda_event for e in iter_events])
        ev = ctypes.addressof(arr)
    _check(_native().cluster_prefill(
        keys, dt, s, n, d, n_clusters, n_iters, init_idx,
        reps, reps.shape[1], unit_start, unit_size, assign, perm,
        values, k_pool, v_pool, pool_rows, int(pool_on_host), ev,
        ws, wsb, stream))


def cluster_prefill_pipelined_workspace_size(slices_per_chunk, n_tokens, n_clusters, dtype_code, pool_on_host,
                                             copy_engine, d=128) -> int:
    return _native().cluster_prefill_pipelined_workspace_size(
        slices_per_chunk, n_tokens, d, n_clusters, dtype_code, int(pool_on_host), int(copy_engine))


def cluster_prefill_pipelined(keys, n_clusters: int, n_iters: int, init_idx, reps, unit_start, unit_size, assign,
                              perm, values, k_pool, v_pool, slices_per_chunk: int, chunk_events: Sequence,
                              copy_stream, pool_on_host: bool = False, copy_engine: bool = True, workspace=None,
                              stream=None):
    """louiskv_cluster_prefill_pipelined: chunk_events holds ceil(S / chunk) + 1
    torch.cuda.Event objects (recorded once already, so that they exist)."""
    s, n, d = keys.shape
    dt = _dtype_code(keys)
    ws, wsb = _ws(workspace, keys.device, cluster_prefill_pipelined_workspace_size, min(slices_per_chunk, s), n,
                  n_clusters, dt, pool_on_host, copy_engine, d)
    arr = (ctypes.c_void_p * len(chunk_events))(*[e.cuda_event for e in chunk_events])
    _check(_native().cluster_prefill_pipelined(
        keys, dt, s, n, d, n_clusters, n_iters, init_idx,
        reps, reps.shape[1], unit_start, unit_size, assign, perm,
        values, k_pool, v_pool, k_pool.shape[1], int(pool_on_host), slices_per_chunk,
        int(copy_engine), ctypes.addressof(arr), len(chunk_events), ws, wsb, stream,
        copy_stream))


def kmeans_assign(keys, n_clusters: int, centroids, assign, workspace=None, stream=None):
    s, n, d = keys.shape
    dt = _dtype_code(keys)
    ws, wsb = _ws(workspace, keys.device, cluster_prefill_workspace_size, s, n, n_clusters, dt, d)
    _check(_native().kmeans_assign(
        keys, dt, s, n, d, n_clusters, centroids, centroids.shape[1], assign,
        ws, wsb, stream))


def kmeans_update(keys, n_clusters: int, assign, centroids_in, centroids_out, counts=None, workspace=None,
                  stream=None):
    s, n, d = keys.shape
    dt = _dtype_code(keys)
    ws, wsb = _ws(workspace, keys.device, cluster_prefill_workspace_size, s, n, n_clusters, dt, d)
    _check(_native().kmeans_update(
        keys, dt, s, n, d, n_clusters, assign, centroids_in, centroids_out,
        centroids_out.shape[1], counts, ws, wsb, stream))


def segment_output(k_new, v_new, k_local, v_local, step: int, seg_len: int, reps, unit_start, unit_size,
                   n_clusters: int, k_pool=None, v_pool=None, prompt_len: int = 0, pool_on_host: bool = False,
                   stream=None):
    s, d = k_new.shape
    pool_rows = k_pool.shape[1] if k_pool is not None else 0
    _check(_native().segment_output(
        k_new, v_new, _dtype_code(k_new), s, d, k_local, v_local, k_local.shape[1],
        step, seg_len, reps, unit_start, unit_size, reps.shape[1], n_clusters,
        k_pool, v_pool, pool_rows, prompt_len, int(pool_on_host), stream))


def boundary_check(q, q_ref, tau: float, mode: int, first_step: bool, fire_out, r_out=None, stream=None):
    g, h, d = q.shape
    _check(_native().boundary_check(
        q, q_ref, _dtype_code(q), g, h, d, float(tau), int(mode), int(first_step),
        r_out, fire_out, stream))


def retrieve_workspace_size(n_slices, units_cap, budget) -> int:
    return _native().retrieve_workspace_size(n_slices, units_cap, budget)


def retrieve(q, n_kv_heads: int, reps, unit_start, unit_size, n_units: int, k_pool, v_pool, budget: int,
             sel_units, n_sel_units, n_sel, k_buf, v_buf, fire=None, scale: Optional[float] = None,
             pool_on_host: bool = False, scores_out=None, workspace=None, stream=None):
    g, hq, d = q.shape
    s = reps.shape[0]
    cap = reps.shape[1]
    ws, wsb = _ws(workspace, q.device, retrieve_workspace_size, s, cap, budget)
    sc = (1.0 / d ** 0.5) if scale is None else scale
    _check(_native().retrieve(
        q, _dtype_code(q), s, n_kv_heads, hq // n_kv_heads, d, float(sc),
        reps, unit_start, unit_size, cap, n_units,
        k_pool, v_pool, k_pool.shape[1], int(pool_on_host), budget, fire,
        sel_units, n_sel_units, n_sel, k_buf, v_buf, scores_out,
        ws, wsb, stream))


def sparse_decode_attn_workspace_size(n_slices, group_size, buf_rows, window, d=128) -> int:
    return _native().sparse_decode_attn_workspace_size(n_slices, group_size, d, buf_rows, window)


def sparse_decode_attn(q, n_kv_heads: int, k_buf, v_buf, n_sel, k_local, v_local, local_start: int, n_local: int,
                       out, lse_out=None, scale: Optional[float] = None, workspace=None, stream=None):
    g, hq, d = q.shape
    s = n_sel.shape[0]
    gs = hq // n_kv_heads
    buf_rows = k_buf.shape[1] if k_buf is not None else 0
    window = k_local.shape[1] if k_local is not None else 0
    ws, wsb = _ws(workspace, q.device, sparse_decode_attn_workspace_size, s, gs, buf_rows, window, d)
    sc = (1.0 / d ** 0.5) if scale is None else scale
    _check(_native().sparse_decode_attn(
        q, _dtype_code(q), s, n_kv_heads, gs, d, float(sc), k_buf, v_buf, n_sel, buf_rows,
        k_local, v_local, window, local_start, n_local, out, _dtype_code(out), lse_out,
        ws, wsb, stream))


def retrieve_rows_workspace_size(n_slices, units_cap) -> int:
    return _native().retrieve_rows_workspace_size(n_slices, units_cap)


def retrieve_rows(q, n_kv_heads: int, reps, unit_start, unit_size, n_units: int, budget: int, sel_units,
                  n_sel_units, n_sel, sel_rows, fire=None, scale: Optional[float] = None, scores_out=None,
                  workspace=None, stream=None):
    """Selection as a list of pool rows (no copy); sel_rows is [S][budget] int32."""
    g, hq, d = q.shape
    s = reps.shape[0]
    cap = reps.shape[1]
    ws, wsb = _ws(workspace, q.device, retrieve_rows_workspace_size, s, cap)
    sc = (1.0 / d ** 0.5) if scale is None else scale
    _check(_native().retrieve_rows(
        q, _dtype_code(q), s, n_kv_heads, hq // n_kv_heads, d, float(sc),
        reps, unit_start, unit_size, cap, n_units, budget, fire,
        sel_units, n_sel_units, n_sel, sel_rows, scores_out,
        ws, wsb, stream))


def sparse_decode_attn_rows_workspace_size(n_slices, group_size, budget, window, d=128) -> int:
    return _native().sparse_decode_attn_rows_workspace_size(n_slices, group_size, d, budget, window)


def sparse_decode_attn_rows(q, n_kv_heads: int, k_pool, v_pool, sel_rows, n_sel, k_local, v_local,
                            local_start: int, n_local: int, out, lse_out=None, scale: Optional[float] = None,
                            workspace=None, stream=None):
    """Attention over the listed pool rows followed by the local window."""
    g, hq, d = q.shape
    s = n_sel.shape[0]
    gs = hq // n_kv_heads
    budget = sel_rows.shape[1]
    window = k_local.shape[1] if k_local is not None else 0
    ws, wsb = _ws(workspace, q.device, sparse_decode_attn_rows_workspace_size, s, gs, budget, window, d)
    sc = (1.0 / d ** 0.5) if scale is None else scale
    _check(_native().sparse_decode_attn_rows(
        q, _dtype_code(q), s, n_kv_heads, gs, d, float(sc), k_pool, v_pool, k_pool.shape[1],
        sel_rows, n_sel, budget, k_local, v_local, window, local_start, n_local,
        out, _dtype_code(out), lse_out, ws, wsb, stream))


def decode_step_workspace_size(n_slices: int, dtype_code: int, group_size: int, units_cap: int, budget: int,
                               window: int) -> int:
    return int(_native().decode_step_workspace_size(n_slices, dtype_code, group_size, units_cap,
                                                                 budget, window))


def decode_step(q, q_ref, tau: float, mode: int, step: int, fire, r_out, k_new, v_new, k_local, v_local,
                seg_len: int, reps, unit_start, unit_size, n_clusters: int, k_pool, v_pool, prompt_len: int,
                budget: int, sel_units, n_sel_units, n_sel, sel_rows, out, lse_out=None, scores_out=None,
                workspace=None, stream=None):
    """One decode step (boundary, store, retrieval of the fired groups, attention)
    in one launch (bf16; two in float32).  workspace: zero-filled before its
    first use."""
    g, hq, d = q.shape
    s = k_new.shape[0]
    h = s // g
    window = k_local.shape[1]
    dt = _dtype_code(q)
    if workspace is None:
        workspace = torch.zeros(decode_step_workspace_size(s, dt, hq // h, reps.shape[1], budget, window),
                                dtype=torch.uint8, device=q.device)
    _check(_native().decode_step(
        q, q_ref, dt, g, hq, h, d, float(tau), mode, step, r_out, fire,
        k_new, v_new, k_local, v_local, window, seg_len, reps, unit_start,
        unit_size, reps.shape[1], n_clusters, k_pool, v_pool, k_pool.shape[1], prompt_len,
        budget, sel_units, n_sel_units, n_sel, sel_rows, scores_out, out,
        _dtype_code(out), lse_out, workspace, workspace.numel(), stream))


def decode_step_cached_workspace_size(n_slices: int, dtype_code: int, group_size: int, units_cap: int, budget: int,
                                      window: int) -> int:
    return int(_native().decode_step_cached_workspace_size(n_slices, dtype_code, group_size, units_cap,
                                                                        budget, window))


def decode_step_cached(q, q_ref, tau: float, mode: int, step: int, fire, r_out, k_new, v_new, k_local, v_local,
                       seg_len: int, reps, unit_start, unit_size, n_clusters: int, k_pool, v_pool, prompt_len: int,
                       budget: int, k_buf, v_buf, buf_row, slot_step, slot_list, sel_units, n_sel_units, n_sel,
                       sel_rows, out, lse_out=None, n_fetched=None, scores_out=None, pool_on_host: bool = False,
                       workspace=None, stream=None):
    """One decode step with KV_critical kept as an LRU cache of k_buf.shape[1]
    pool rows, in four launches.  workspace: zero-filled before its first use."""
    g, hq, d = q.shape
    s = k_new.shape[0]
    h = s // g
    window = k_local.shape[1]
    dt = _dtype_code(q)
    if workspace is None:
        workspace = torch.zeros(decode_step_cached_workspace_size(s, dt, hq // h, reps.shape[1], budget, window),
                                dtype=torch.uint8, device=q.device)
    _check(_native().decode_step_cached(
        q, q_ref, dt, g, hq, h, d, float(tau), mode, step, r_out, fire,
        k_new, v_new, k_local, v_local, window, seg_len, reps, unit_start,
        unit_size, reps.shape[1], n_clusters, k_pool, v_pool, k_pool.shape[1], int(pool_on_host),
        prompt_len, budget, k_buf.shape[1], k_buf, v_buf, buf_row, slot_step,
        slot_list, n_fetched, sel_units, n_sel_units, n_sel, sel_rows,
        scores_out, out, _dtype_code(out), lse_out, workspace, workspace.numel(),
        stream))


NOALLOC_SCRATCH_BYTES = 8 << 20   # LOUISKV_NOALLOC_SCRATCH_BYTES


def sparse_decode_attn_rows_noalloc(q, n_kv_heads: int, k_pool, v_pool, sel_rows, n_sel, k_local, v_local,
                                    local_start: int, n_local: int, out, lse_out=None,
                                    scale: Optional[float] = None, stream=None):
    """sparse_decode_attn_rows without a workspace: the split-KV partials use
    the library's static device array (at most NOALLOC_SCRATCH_BYTES)."""
    g, hq, d = q.shape
    s = n_sel.shape[0]
    gs = hq // n_kv_heads
    budget = sel_rows.shape[1]
    window = k_local.shape[1] if k_local is not None else 0
    sc = (1.0 / d ** 0.5) if scale is None else scale
    _check(_native().sparse_decode_attn_rows_noalloc(
        q, _dtype_code(q), s, n_kv_heads, gs, d, float(sc), k_pool, v_pool, k_pool.shape[1],
        sel_rows, n_sel, budget, k_local, v_local, window, local_start, n_local,
        out, _dtype_code(out), lse_out, stream))


def decode_prologue(q, q_ref, tau: float, mode: int, first_step: bool, fire, r_out, k_new, v_new, k_local, v_local,
                    step: int, seg_len: int, reps, unit_start, unit_size, n_clusters: int, k_pool=None, v_pool=None,
                    prompt_len: int = 0, pool_on_host: bool = False, stream=None):
    """boundary_check and segment_output (fixed segments) in one launch."""
    g, hq, d = q.shape
    s = k_new.shape[0]
    window = k_local.shape[1]
    pool_rows = k_pool.shape[1] if k_pool is not None else 0
    _check(_native().decode_prologue(
        q, q_ref, _dtype_code(q), g, hq, d, float(tau), mode, int(first_step), r_out, fire,
        k_new, v_new, s, k_local, v_local, window, step, seg_len, reps,
        unit_start, unit_size, reps.shape[1], n_clusters, k_pool, v_pool, pool_rows,
        prompt_len, int(pool_on_host), stream))


# ------------------------------------------------------ ablation baselines

def fire_every(fire, step: int, stride: int, stream=None):
    """Fixed-stride trigger: fire[g] = (step % stride == 0) for every group."""
    _check(_native().fire_every(fire, fire.shape[0], step, stride, stream))


def page_prefill(keys, page_len: int, reps, unit_start, unit_size, values=None, k_pool=None, v_pool=None,
                 pool_on_host: bool = False, stream=None):
    """Page-level index of the prompt (mean key per page), pool in token order."""
    s, n, d = keys.shape
    pool_rows = k_pool.shape[1] if k_pool is not None else 0
    _check(_native().page_prefill(
        keys, values, _dtype_code(keys), s, n, d, page_len, reps, reps.shape[1],
        unit_start, unit_size, k_pool, v_pool, pool_rows, int(pool_on_host),
        stream))


def retrieve_rows_per_head(q, n_kv_heads: int, reps, unit_start, unit_size, n_units: int, budget: int, sel_units,
                           n_sel_units, n_sel, sel_rows, fire=None, scale: Optional[float] = None, scores_out=None,
                           workspace=None, stream=None):
    """One selection per query head; outputs have n_slices * group_size lists."""
    g, hq, d = q.shape
    s = reps.shape[0]
    cap = reps.shape[1]
    gs = hq // n_kv_heads
    ws, wsb = _ws(workspace, q.device, retrieve_rows_workspace_size, s * gs, cap)
    sc = (1.0 / d ** 0.5) if scale is None else scale
    _check(_native().retrieve_rows_per_head(
        q, _dtype_code(q), s, n_kv_heads, gs, d, float(sc),
        reps, unit_start, unit_size, cap, n_units, budget, fire,
        sel_units, n_sel_units, n_sel, sel_rows, scores_out,
        ws, wsb, stream))


def sparse_decode_attn_rows_per_head(q, n_kv_heads: int, k_pool, v_pool, sel_rows, n_sel, k_local, v_local,
                                     local_start: int, n_local: int, out, lse_out=None, scale: Optional[float] = None,
                                     workspace=None, stream=None):
    """Attention of every query head over its own listed pool rows and its KV
    head's local window."""
    g, hq, d = q.shape
    s = k_pool.shape[0]
    gs = hq // n_kv_heads
    budget = sel_rows.shape[1]
    window = k_local.shape[1] if k_local is not None else 0
    ws, wsb = _ws(workspace, q.device, sparse_decode_attn_rows_workspace_size, s * gs, 1, budget, window, d)
    sc = (1.0 / d ** 0.5) if scale is None else scale
    _check(_native().sparse_decode_attn_rows_per_head(
        q, _dtype_code(q), s, n_kv_heads, gs, d, float(sc), k_pool, v_pool, k_pool.shape[1],
        sel_rows, n_sel, budget, k_local, v_local, window, local_start, n_local,
        out, _dtype_code(out), lse_out, ws, wsb, stream))


# ------------------------------------------------ boundary-delimited segments

def segment_state_ints(window: int) -> int:
    """int32 entries per slice of the segment state (louiskv_segment_state_ints)."""
    return _native().segment_state_ints(window)


def segment_state_init(seg_state, window: int, n_clusters: int, stream=None):
    """Segment state before decode step 0 (clusters only, empty window)."""
    _check(_native().segment_state_init(seg_state, seg_state.shape[0], window, n_clusters,
                                                     stream))


def segment_output_boundary(k_new, v_new, k_local, v_local, step: int, seg_max: int, fire, seg_state, reps,
                            unit_start, unit_size, n_clusters: int, n_kv_heads: int, k_pool=None, v_pool=None,
                            prompt_len: int = 0, pool_on_host: bool = False, stream=None):
    s, d = k_new.shape
    pool_rows = k_pool.shape[1] if k_pool is not None else 0
    _check(_native().segment_output_boundary(
        k_new, v_new, _dtype_code(k_new), s, n_kv_heads, d, k_local, v_local,
        k_local.shape[1], step, seg_max, fire, seg_state, reps, unit_start,
        unit_size, reps.shape[1], n_clusters, k_pool, v_pool, pool_rows, prompt_len,
        int(pool_on_host), stream))


def retrieve_seg(q, n_kv_heads: int, reps, unit_start, unit_size, max_units: int, seg_state, window: int, k_pool,
                 v_pool, budget: int, sel_units, n_sel_units, n_sel, k_buf, v_buf, fire=None,
                 scale: Optional[float] = None, pool_on_host: bool = False, scores_out=None, workspace=None,
                 stream=None):
    g, hq, d = q.shape
    s = reps.shape[0]
    cap = reps.shape[1]
    ws, wsb = _ws(workspace, q.device, retrieve_workspace_size, s, cap, budget)
    sc = (1.0 / d ** 0.5) if scale is None else scale
    _check(_native().retrieve_seg(
        q, _dtype_code(q), s, n_kv_heads, hq // n_kv_heads, d, float(sc),
        reps, unit_start, unit_size, cap, max_units, seg_state, window,
        k_pool, v_pool, k_pool.shape[1], int(pool_on_host), budget, fire,
        sel_units, n_sel_units, n_sel, k_buf, v_buf, scores_out,
        ws, wsb, stream))


def retrieve_rows_seg(q, n_kv_heads: int, reps, unit_start, unit_size, max_units: int, seg_state, window: int,
                      budget: int, sel_units, n_sel_units, n_sel, sel_rows, fire=None, scale: Optional[float] = None,
                      scores_out=None, workspace=None, stream=None):
    g, hq, d = q.shape
    s = reps.shape[0]
    cap = reps.shape[1]
    ws, wsb = _ws(workspace, q.device, retrieve_rows_workspace_size, s, cap)
    sc = (1.0 / d ** 0.5) if scale is None else scale
    _check(_native().retrieve_rows_seg(
        q, _dtype_code(q), s, n_kv_heads, hq // n_kv_heads, d, float(sc),
        reps, unit_start, unit_size, cap, max_units, seg_state, window, budget,
        fire, sel_units, n_sel_units, n_sel, sel_rows, scores_out,
        ws, wsb, stream))


def sparse_decode_attn_seg(q, n_kv_heads: int, k_buf, v_buf, n_sel, k_local, v_local, seg_state, n_tokens: int,
                           out, lse_out=None, scale: Optional[float] = None, workspace=None, stream=None):
    g, hq, d = q.shape
    s = n_sel.shape[0]
    gs = hq // n_kv_heads
    buf_rows = k_buf.shape[1] if k_buf is not None else 0
    window = k_local.shape[1]
    ws, wsb = _ws(workspace, q.device, sparse_decode_attn_workspace_size, s, gs, buf_rows, window, d)
    sc = (1.0 / d ** 0.5) if scale is None else scale
    _check(_native().sparse_decode_attn_seg(
        q, _dtype_code(q), s, n_kv_heads, gs, d, float(sc), k_buf, v_buf, n_sel, buf_rows,
        k_local, v_local, window, seg_state, n_tokens, out, _dtype_code(out),
        lse_out, ws, wsb, stream))


def sparse_decode_attn_rows_seg(q, n_kv_heads: int, k_pool, v_pool, sel_rows, n_sel, k_local, v_local, seg_state,
                                n_tokens: int, out, lse_out=None, scale: Optional[float] = None, workspace=None,
                                stream=None):
    g, hq, d = q.shape
    s = n_sel.shape[0]
    gs = hq // n_kv_heads
    budget = sel_rows.shape[1]
    window = k_local.shape[1]
    ws, wsb = _ws(workspace, q.device, sparse_decode_attn_rows_workspace_size, s, gs, budget, window, d)
    sc = (1.0 / d ** 0.5) if scale is None else scale
    _check(_native().sparse_decode_attn_rows_seg(
        q, _dtype_code(q), s, n_kv_heads, gs, d, float(sc), k_pool, v_pool, k_pool.shape[1],
        sel_rows, n_sel, budget, k_local, v_local, window, seg_state, n_tokens,
        out, _dtype_code(out), lse_out, ws, wsb, stream))


def retrieve_delta_workspace_size(n_slices, units_cap, budget) -> int:
    return _native().retrieve_delta_workspace_size(n_slices, units_cap, budget)


def retrieve_delta(q, n_kv_heads: int, reps, unit_start, unit_size, n_units: int, k_pool, v_pool, budget: int,
                   sel_units, n_sel_units, n_sel, k_buf, v_buf, buf_row, slot_list, fire=None, seg_state=None,
                   window: int = 0, n_fetched=None, scale: Optional[float] = None, pool_on_host: bool = False,
                   scores_out=None, workspace=None, stream=None):
    """Retrieval into KV_critical as a cache of pool rows (only new rows are copied)."""
    g, hq, d = q.shape
    s = reps.shape[0]
    cap = reps.shape[1]
    ws, wsb = _ws(workspace, q.device, retrieve_delta_workspace_size, s, cap, budget)
    sc = (1.0 / d ** 0.5) if scale is None else scale
    _check(_native().retrieve_delta(
        q, _dtype_code(q), s, n_kv_heads, hq // n_kv_heads, d, float(sc),
        reps, unit_start, unit_size, cap, n_units, seg_state, window,
        k_pool, v_pool, k_pool.shape[1], int(pool_on_host), budget, fire,
        sel_units, n_sel_units, n_sel, k_buf, v_buf, buf_row,
        slot_list, n_fetched, scores_out, ws, wsb, stream))


CACHE_MAX_ROWS = 65536   # louiskv_retrieve_cached: slots per slice at most


def retrieve_cached(q, n_kv_heads: int, reps, unit_start, unit_size, n_units: int, k_pool, v_pool, budget: int,
                    step: int, sel_units, n_sel_units, n_sel, k_buf, v_buf, buf_row, slot_step, slot_list, fire=None,
                    seg_state=None, window: int = 0, n_fetched=None, scale: Optional[float] = None,
                    pool_on_host: bool = False, scores_out=None, workspace=None, stream=None):
    """Retrieval into KV_critical kept as an LRU cache of k_buf.shape[1] pool rows."""
    g, hq, d = q.shape
    s = reps.shape[0]
    cap = reps.shape[1]
    ws, wsb = _ws(workspace, q.device, retrieve_delta_workspace_size, s, cap, budget)
    sc = (1.0 / d ** 0.5) if scale is None else scale
    _check(_native().retrieve_cached(
        q, _dtype_code(q), s, n_kv_heads, hq // n_kv_heads, d, float(sc),
        reps, unit_start, unit_size, cap, n_units, seg_state, window,
        k_pool, v_pool, k_pool.shape[1], int(pool_on_host), budget, k_buf.shape[1], step, fire,
        sel_units, n_sel_units, n_sel, k_buf, v_buf, buf_row, slot_step,
        slot_list, n_fetched, scores_out, ws, wsb, stream))


def pack_pool(keys, values, perm, k_pool, v_pool=None, pool_on_host: bool = False, stream=None):
    """Prompt K/V rows into the pools in perm order (each cluster contiguous)."""
    s, n, d = keys.shape
    _check(_native().pack_pool(
        keys, values, _dtype_code(keys), s, n, d, perm, k_pool, v_pool,
        k_pool.shape[1], int(pool_on_host), stream))
