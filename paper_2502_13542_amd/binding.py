"""Thin binding of libactqkv.so: same names as the C ABI, argument marshalling only
(in _native, built from csrc/py_native.cpp; load_library() gives the plain ctypes
view of the library).  Tensors are torch tensors on the GPU (torch is used for
device memory and streams, nothing else); every step runs in the library's
kernels.  There is no fallback: if the library is missing or a call fails, an
exception is raised.
"""
from __future__ import annotations

import ctypes
import importlib
import os
from typing import Optional

import torch

from .synth import LayerShape

_HERE = os.path.dirname(os.path.abspath(__file__))
LIB_PATH = os.path.join(_HERE, "libactqkv.so")
NATIVE_PATH = os.path.join(_HERE, "_native.so")

ACTQKV_F32, ACTQKV_BF16 = 0, 1
STATS_UPDATE, PROBE_MEAN_POOLING, PROBE_WINDOW_CHAIN = 1, 2, 4   # bits of build_probe's update_stats
SELECT_ENTROPY_TOPK = 1                                          # bit of select's flags
DECODE_SCORES_ONLY = 2                                           # bit of decode_retrieve's flags
DECODE_NO_WAIT = 4                                               # bit of decode_layer's flags
SELECT_DENSITY_ONLY, SELECT_GIVEN_COUNT = 8, 16                  # bits of select's flags
ERROR_NAMES = {0: "OK", -1: "EINVAL", -2: "ESHAPE", -3: "EALIGN", -4: "EWORKSPACE", -5: "EHIP"}


class ActQKVError(RuntimeError):
    def __init__(self, code: int, message: str):
        super().__init__(f"actqkv error {ERROR_NAMES.get(code, code)}: {message}")
        self.code = code


class CShape(ctypes.Structure):
    _fields_ = [("n_q_heads", ctypes.c_int32), ("n_kv_heads", ctypes.c_int32),
                ("head_dim", ctypes.c_int32), ("block_size", ctypes.c_int32),
                ("n_rep", ctypes.c_int32), ("n_init", ctypes.c_int32),
                ("n_local", ctypes.c_int32), ("dtype", ctypes.c_int32),
                ("softmax_scale", ctypes.c_float), ("var_eps", ctypes.c_float)]


def c_shape(s: LayerShape, softmax_scale: float = 0.0, var_eps: float = 0.0) -> CShape:
    return CShape(s.n_q_heads, s.n_kv_heads, s.head_dim, s.block_size, s.n_rep, s.n_init,
                  s.n_local, ACTQKV_F32 if s.dtype == "fp32" else ACTQKV_BF16,
                  softmax_scale, var_eps)


_lib = None
_native = None      # the extension module, once load_library has run

_vp, _i, _i64, _sz = ctypes.c_void_p, ctypes.c_int, ctypes.c_int64, ctypes.c_size_t
_shp = ctypes.POINTER(CShape)
SIGNATURES = {
    "actqkv_stats_floats": (_sz, [_shp]),
    "actqkv_workspace_bytes": (_sz, [_shp, _i, _i, _i, _i]),
    "actqkv_build_probe": (_i, [_shp, _i, _i, _vp, _vp, _i, _vp, _vp, _vp, _vp, _vp, _sz, _vp]),
    "actqkv_score_blocks": (_i, [_shp, _i, _vp, _vp, _vp, _i64, _i, _i, _vp, _vp, _i64, _vp]),
    "actqkv_select": (_i, [_i, _vp, _i64, _i, _i, _vp, _i, _i, _vp, _vp, _vp, _vp, _vp, _vp, _vp]),
    "actqkv_retrieval_attention": (_i, [_shp, _i, _i, _vp, _vp, _vp, _i64, _i, _vp, _vp, _vp, _i,
                                        _vp, _vp, _vp, _sz, _vp]),
    "actqkv_retrieval_attention_static": (_i, [_shp, _i, _i, _vp, _vp, _vp, _i64, _i, _vp, _vp, _vp, _i,
                                               _vp, _vp, _vp]),
    "actqkv_retrieval_attention_per_head": (_i, [_shp, _i, _i, _vp, _vp, _vp, _i64, _i, _vp, _vp, _vp, _i,
                                                 _vp, _vp, _vp, _sz, _vp]),
    "actqkv_score_blocks_per_head": (_i, [_shp, _i, _vp, _vp, _i64, _i, _i, _vp, _vp, _i64, _vp]),
    "actqkv_append_kv": (_i, [_shp, _i, _i, _vp, _vp, _vp, _vp, _vp, _i64, _vp, _i64, _i, _vp]),
    "actqkv_cutoff_budgets": (_i, [_i, _i, ctypes.c_float, _i, _vp, _vp, _vp, _vp, _vp]),
    "actqkv_cutoff_next_step": (_i, [_i, _i, ctypes.c_float, ctypes.c_float, _vp, _vp, _vp, _vp, _vp, _vp]),
    "actqkv_append_kv_probe": (_i, [_shp, _i, _vp, _vp, _vp, _vp, _vp, _vp, _i64, _vp, _i64, _i, _vp, _vp, _vp, _vp]),
    "actqkv_decode_retrieve": (_i, [_shp, _i, _vp, _vp, _vp, _vp, _vp, _vp, _i64, _vp, _i64, _i, _i, _vp, _vp, _vp,
                                    _vp, _vp, _i64, _i, _i, _vp, _vp, _vp, _vp, _vp, _vp, _vp]),
    "actqkv_decode_select_attention": (_i, [_shp, _i, _vp, _vp, _vp, _i64, _i, _vp, _vp, _i64, _i, _vp, _i, _i,
                                            _vp, _vp, _vp, _vp, _vp, _vp, _vp, _vp, _vp, _vp, _sz, _vp]),
    "actqkv_decode_layer": (_i, [_shp, _i, _vp, _vp, _vp, _vp, _vp, _i64, _vp, _i64, _i, _vp, _i, _vp, _vp, _i64, _i,
                                 _i, _vp, _vp, _vp, _vp, _vp, _vp, _vp, _vp, _vp, _vp, _sz, _vp]),
    "actqkv_retrieval_attention_teams": (_i, [_shp, _i, _i, _vp, _vp, _vp, _i64, _i, _vp, _vp, _vp, _i,
                                              _vp, _vp, _vp, _sz, _i, _i, _vp, _vp]),
    "actqkv_window_step": (_i, [_shp, _i, _i, _vp, _vp, _i, _vp, _vp, _vp, _vp, _vp, _i64, _i, _i, _vp, _vp, _i64, _i, _i, _vp,
                                _vp, _vp, _vp, _vp, _vp, _vp, _vp, _i64, _i, _vp, _vp, _vp, _vp, _sz, _vp]),
    "actqkv_decode_step": (_i, [_shp, _i, _vp, _vp, _vp, _vp, _vp, _vp, _i64, _vp, _i64, _i, _i, _vp, _vp, _vp, _vp, _vp, _i64,
                                _i, _i, _vp, _vp, _vp, _vp, _vp, _vp, _i, _vp, _vp, _vp, _vp, _sz, _vp]),
    "actqkv_copy_bytes": (_i, [_vp, _vp, _sz, _vp]),
    "actqkv_gather_blocks": (_i, [_shp, _i, _vp, _vp, _i64, _i, _vp, _vp, _i, _vp, _vp, _i64, _i, _i, _vp, _vp]),
    "actqkv_gather_blocks_cached": (_i, [_shp, _i, _vp, _vp, _i, _vp, _vp, _i, _vp, _vp, _i, _i, _i, _i, _i, _i, _i,
                                         _i, _i, _i, _vp, _vp, _vp]),
    "actqkv_retrieval_attention_windows": (_i, [_shp, _i, _i, _vp, _vp, _vp, _i, _vp, _vp, _vp, _i, _vp, _vp, _vp, _sz,
                                                _i, _vp]),
    "actqkv_last_error": (ctypes.c_char_p, []),
    "actqkv_prefill_cut": (_i, [_shp, _i, _i, _i, _i, _vp]),
    "actqkv_version": (_i, []),
}


def load_library(build_if_missing: bool = True) -> ctypes.CDLL:
    """Loads libactqkv.so and the extension module that calls it (building them first if they have
    never been built)."""
    global _lib, _native
    if _lib is not None:
        return _lib
    path = os.environ.get("ACTQKV_LIB") or LIB_PATH    # another build of the library, for comparisons
    missing = [p for p in (path, NATIVE_PATH) if p in (LIB_PATH, NATIVE_PATH) and not os.path.exists(p)]
    if missing:
        if not build_if_missing:
            raise FileNotFoundError(missing[0])
        from .build import build
        build()
    lib = ctypes.CDLL(path)
    for name, (res, args) in SIGNATURES.items():
        if path != LIB_PATH and not hasattr(lib, name):
            continue               # an older build: a call of what it lacks raises (LayerRunner needs actqkv_window_step, actqkv_decode_step)
        fn = getattr(lib, name)
        fn.restype, fn.argtypes = res, args
    native = importlib.import_module("._native", __package__)
    native.load(path, ActQKVError)
    _lib, _native = lib, native
    return lib


def _calls():
    """The extension module."""
    if _native is None:
        load_library()
    return _native


def _check(rc: int) -> None:
    if rc != 0:
        raise ActQKVError(rc, load_library().actqkv_last_error().decode())


def _ptr_readable(t: torch.Tensor, dtype=None) -> int:
    """A tensor a kernel may read in place: device memory or pinned host memory.  (The runtime is asked each
    time: an address that was pinned once may belong to pageable memory by now.)"""
    if not (t.is_cuda or t.is_pinned()):
        raise ActQKVError(-1, "tensor is neither on the GPU nor in pinned host memory")
    if not t.is_contiguous():
        raise ActQKVError(-1, "tensor is not contiguous")
    if dtype is not None and t.dtype != dtype:
        raise ActQKVError(-1, f"tensor dtype {t.dtype}, expected {dtype}")
    return t.data_ptr()


def version() -> int:
    return load_library().actqkv_version()


def last_error() -> str:
    return load_library().actqkv_last_error().decode()


def stats_floats(shape: CShape) -> int:
    return load_library().actqkv_stats_floats(ctypes.byref(shape))


def workspace_bytes(shape: CShape, batch: int, m: int, nb_capacity: int, k_cap: int) -> int:
    n = load_library().actqkv_workspace_bytes(ctypes.byref(shape), batch, m, nb_capacity, k_cap)
    if n == 0:
        raise ActQKVError(-1, last_error())
    return n


def prefill_cut(shape: CShape, batch: int, m: int, k_cap: int, cus: int = 256) -> tuple:
    """(rows of a workgroup, query tiles, pieces altogether, merged by a launch) of an attention call; see the header."""
    cut = (ctypes.c_int32 * 4)()
    if load_library().actqkv_prefill_cut(ctypes.byref(shape), batch, m, k_cap, cus, cut) != 0:
        raise ActQKVError(-1, last_error())
    return tuple(cut)


def append_kv(shape: CShape, batch: int, m: int, k_new, v_new, pos0, k_cache, v_cache,
              cache_seq_stride: int, rep_keys, rep_seq_stride: int, nb_capacity: int, stream=None) -> None:
    _calls().append_kv(shape, batch, m, k_new, v_new, pos0, k_cache, v_cache, cache_seq_stride, rep_keys,
                       rep_seq_stride, nb_capacity, stream)


def append_kv_probe(shape: CShape, batch: int, q_tok, k_new, v_new, pos0, k_cache, v_cache,
                    cache_seq_stride: int, rep_keys, rep_seq_stride: int, nb_capacity: int, probe, probe_kv,
                    probe_norm, stream=None) -> None:
    _calls().append_kv_probe(shape, batch, q_tok, k_new, v_new, pos0, k_cache, v_cache, cache_seq_stride, rep_keys,
                             rep_seq_stride, nb_capacity, probe, probe_kv, probe_norm, stream)


def window_step(shape: CShape, batch: int, m: int, q_win, stats, update_stats: int, probe, probe_kv, probe_norm, weights,
                rep_keys, rep_seq_stride: int, nb_scored: int, nb_begin: int, nb_end, scores, score_stride: int, k_cap: int,
                budget_remaining, theta_rest_sum, idx, n_sel, theta, budget, k_cache, v_cache, cache_seq_stride: int,
                nb_capacity: int, n_ctx, out, lse, workspace, stream=None, flags: int = 0) -> None:
    """Probe, scores, selection and attention of a window in one call; see the header."""
    _calls().window_step(shape, batch, m, q_win, stats, int(update_stats), probe, probe_kv, probe_norm, weights, rep_keys,
                         rep_seq_stride, nb_scored, nb_begin, nb_end, scores, score_stride, k_cap, int(flags),
                         budget_remaining, theta_rest_sum, idx, n_sel, theta, budget, k_cache, v_cache, cache_seq_stride,
                         nb_capacity, n_ctx, out, lse, workspace, stream)


def decode_step(shape: CShape, batch: int, q_tok, k_new, v_new, pos0, k_cache, v_cache, cache_seq_stride: int, rep_keys,
                rep_seq_stride: int, nb_scored: int, nb_begin: int, nb_end, probe, probe_kv, probe_norm, scores,
                score_stride: int, k_cap: int, budget_remaining, theta_rest_sum, idx, n_sel, theta, budget, nb_capacity: int,
                n_ctx, out, lse, workspace, stream=None, flags: int = 0) -> None:
    """Cache update, probe, scores, selection and attention of a decode step in one call; see the header."""
    _calls().decode_step(shape, batch, q_tok, k_new, v_new, pos0, k_cache, v_cache, cache_seq_stride, rep_keys, rep_seq_stride,
                         nb_scored, nb_begin, nb_end, probe, probe_kv, probe_norm, scores, score_stride, k_cap, int(flags),
                         budget_remaining, theta_rest_sum, idx, n_sel, theta, budget, nb_capacity, n_ctx, out, lse, workspace,
                         stream)


def decode_retrieve(shape: CShape, batch: int, q_tok, k_new, v_new, pos0, k_cache, v_cache,
                    cache_seq_stride: int, rep_keys, rep_seq_stride: int, nb_capacity: int, nb_begin: int,
                    nb_end, probe, probe_kv, probe_norm, scores, score_stride: int, k_cap: int,
                    budget_remaining, theta_rest_sum, idx, n_sel, theta, budget, stream=None,
                    flags: int = 0) -> None:
    """Cache update, probe, scores and selection of a decode step in one call; see the header."""
    _calls().decode_retrieve(shape, batch, q_tok, k_new, v_new, pos0, k_cache, v_cache, cache_seq_stride, rep_keys,
                             rep_seq_stride, nb_capacity, nb_begin, nb_end, probe, probe_kv, probe_norm, scores,
                             score_stride, k_cap, int(flags), budget_remaining, theta_rest_sum, idx, n_sel, theta,
                             budget, stream)


def decode_select_attention(shape: CShape, batch: int, q, k_cache, v_cache, seq_stride: int, nb_capacity: int,
                            n_ctx, scores, score_stride: int, nb_begin: int, nb_end, k_cap: int, budget_in,
                            theta_rest_sum, budget_after, idx, n_sel, theta, budget, out, lse, workspace,
                            stream=None, flags: int = 0) -> None:
    """Selection and attention of a decode step in one launch; see the header."""
    _calls().decode_select_attention(shape, batch, q, k_cache, v_cache, seq_stride, nb_capacity, n_ctx, scores,
                                     score_stride, nb_begin, nb_end, k_cap, int(flags), budget_in, theta_rest_sum,
                                     budget_after, idx, n_sel, theta, budget, out, lse, workspace, stream)


def decode_layer(shape: CShape, batch: int, q, k_new, v_new, k_cache, v_cache, cache_seq_stride: int,
                 rep_keys, rep_seq_stride: int, nb_capacity: int, n_ctx, nb_begin: int, nb_end, scores,
                 score_stride: int, k_cap: int, budget_in, theta_rest_sum, budget_after, idx, n_sel, theta,
                 budget, out, lse, workspace, stream=None, flags: int = 0) -> None:
    """A whole layer of a decode step in one launch; see the header."""
    _calls().decode_layer(shape, batch, q, k_new, v_new, k_cache, v_cache, cache_seq_stride, rep_keys, rep_seq_stride,
                          nb_capacity, n_ctx, nb_begin, nb_end, scores, score_stride, k_cap, int(flags), budget_in,
                          theta_rest_sum, budget_after, idx, n_sel, theta, budget, out, lse, workspace, stream)


def retrieval_attention_static(shape: CShape, batch: int, m: int, q, k_cache, v_cache, seq_stride: int,
                               nb_capacity: int, n_ctx, idx, n_sel, k_cap: int, out, lse, stream=None) -> None:
    """The attention with the library's own scratch array instead of a workspace; see the header."""
    _calls().retrieval_attention_static(shape, batch, m, q, k_cache, v_cache, seq_stride, nb_capacity, n_ctx, idx,
                                        n_sel, k_cap, out, lse, stream)


def retrieval_attention_teams(shape: CShape, batch: int, m: int, q, k_cache, v_cache, seq_stride: int,
                              nb_capacity: int, n_ctx, idx, n_sel, k_cap: int, out, lse, workspace,
                              first_cus: int, late_cus: int, stream=None, stream_late=None) -> None:
    """The attention on first_cus compute units, with an optional second team of late_cus workgroups
    launched on stream_late; see the header."""
    _calls().retrieval_attention_teams(shape, batch, m, q, k_cache, v_cache, seq_stride, nb_capacity, n_ctx, idx,
                                       n_sel, k_cap, out, lse, workspace, int(first_cus), int(late_cus), stream,
                                       stream_late)


def retrieval_attention_windows(shape: CShape, n_windows: int, m: int, q, k_cache, v_cache, nb_capacity: int, n_ctx,
                                idx, n_sel, k_cap: int, out, lse, workspace, cus: int = 256, stream=None) -> None:
    """The attention of several windows of one sequence in one launch, each as if alone; see the header."""
    _calls().retrieval_attention_windows(shape, n_windows, m, q, k_cache, v_cache, nb_capacity, n_ctx, idx, n_sel, k_cap,
                                         out, lse, workspace, cus, stream)


def cutoff_budgets(batch: int, n_layers: int, k_mean: float, k_cap: int, theta, budget, count, budget_left=None,
                   stream=None) -> None:
    _calls().cutoff_budgets(batch, n_layers, k_mean, k_cap, theta, budget, count, budget_left, stream)


def cutoff_next_step(batch: int, n_layers: int, k_mean: float, theta_prior: float, theta_prev,
                     theta_sum, n_steps, budget_remaining, theta_rest_sum, stream=None) -> None:
    _calls().cutoff_next_step(batch, n_layers, k_mean, theta_prior, theta_prev, theta_sum, n_steps, budget_remaining,
                              theta_rest_sum, stream)


def copy_bytes(dst, src, stream=None) -> None:
    """Plain copy of src into dst by one kernel; either may be device memory or pinned host memory."""
    n = src.numel() * src.element_size()
    if dst.numel() * dst.element_size() != n:
        raise ActQKVError(-1, "copy_bytes: sizes differ")
    _calls().copy_bytes(_ptr_readable(dst), _ptr_readable(src), n, stream)


def copy_bytes_at(dst, dst_byte: int, src, src_byte: int, n_bytes: int, stream=None) -> None:
    """copy_bytes between byte offsets of two tensors, without making views of them (a slice costs
    the host about as much as the launch); offsets and length are checked against the tensors."""
    if dst_byte < 0 or src_byte < 0 or n_bytes < 0 or dst_byte + n_bytes > dst.numel() * dst.element_size() \
            or src_byte + n_bytes > src.numel() * src.element_size():
        raise ActQKVError(-1, "copy_bytes_at: range outside a tensor")
    _calls().copy_bytes(_ptr_readable(dst) + dst_byte, _ptr_readable(src) + src_byte, n_bytes, stream)


def build_probe(shape: CShape, batch: int, m: int, q_win, stats, update_stats, probe, probe_kv,
                probe_norm, weights, workspace, stream=None) -> None:
    _calls().build_probe(shape, batch, m, q_win, stats, int(update_stats), probe, probe_kv, probe_norm, weights,
                         workspace, stream)


def gather_blocks(shape: CShape, batch: int, k_store, v_store, store_seq_stride: int, nb_store: int,
                  idx, n_sel, k_cap: int, k_cache, v_cache, cache_seq_stride: int, nb_capacity: int,
                  slot0: int, idx_slots, stream=None) -> None:
    _calls().gather_blocks(shape, batch, k_store, v_store, store_seq_stride, nb_store, idx, n_sel, k_cap, k_cache,
                           v_cache, cache_seq_stride, nb_capacity, slot0, idx_slots, stream)


def gather_blocks_cached(shape: CShape, n_windows: int, k_store, v_store, nb_store: int, idx, n_sel, k_cap: int,
                         k_cache, v_cache, nb_capacity: int, slot0: int, n_slots: int, here0, here1, group: int, state,
                         idx_slots, stream=None) -> None:
    """The blocks a group of windows selects into slots that keep their blocks; here0, here1: (lo, hi, at)
    of blocks that lie in the cache itself.  See the header."""
    _calls().gather_blocks_cached(shape, n_windows, k_store, v_store, nb_store, idx, n_sel, k_cap, k_cache, v_cache,
                                  nb_capacity, slot0, n_slots, *here0, *here1, group, state, idx_slots, stream)


def score_blocks(shape: CShape, batch: int, probe_kv, probe_norm, rep_keys, seq_stride: int,
                 nb_capacity: int, nb_begin: int, nb_end, scores, score_stride: int,
                 stream=None) -> None:
    _calls().score_blocks(shape, batch, probe_kv, probe_norm, rep_keys, seq_stride, nb_capacity, nb_begin, nb_end,
                          scores, score_stride, stream)


def score_blocks_per_head(shape: CShape, batch: int, probe, rep_keys, seq_stride: int, nb_capacity: int,
                          nb_begin: int, nb_end, scores, score_stride: int, stream=None) -> None:
    _calls().score_blocks_per_head(shape, batch, probe, rep_keys, seq_stride, nb_capacity, nb_begin, nb_end, scores,
                                   score_stride, stream)


def select(batch: int, scores, score_stride: int, nb_capacity: int, nb_begin: int, nb_end,
           k_cap: int, budget_remaining, theta_rest_sum, idx, n_sel, theta=None, budget=None,
           stream=None, flags: int = 0) -> None:
    _calls().select(batch, scores, score_stride, nb_capacity, nb_begin, nb_end, k_cap, int(flags), budget_remaining,
                    theta_rest_sum, idx, n_sel, theta, budget, stream)


def retrieval_attention(shape: CShape, batch: int, m: int, q, k_cache, v_cache, seq_stride: int,
                        nb_capacity: int, n_ctx, idx, n_sel, k_cap: int, out, lse, workspace,
                        stream=None, per_head: bool = False) -> None:
    """per_head: idx [batch][Hk][k_cap], n_sel [batch][Hk] (actqkv_retrieval_attention_per_head)."""
    attend = _calls().retrieval_attention_per_head if per_head else _calls().retrieval_attention
    attend(shape, batch, m, q, k_cache, v_cache, seq_stride, nb_capacity, n_ctx, idx, n_sel, k_cap, out, lse,
           workspace, stream)
