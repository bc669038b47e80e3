"""ctypes loader for libcake.so.  Fails loudly when the library has not been built."""
from __future__ import annotations

import ctypes
import os

LIB_PATH = os.path.join(os.path.dirname(os.path.abspath(__file__)), "libcake.so")


class cake_shape(ctypes.Structure):
    _fields_ = [(n, ctypes.c_int32) for n in
                ("batch", "n_layers", "n_q_heads", "n_kv_heads", "head_dim", "seq_len", "window", "dtype")]


class cake_params(ctypes.Structure):
    _fields_ = [("scale", ctypes.c_float), ("gamma", ctypes.c_float), ("tau1", ctypes.c_float),
                ("tau2", ctypes.c_float), ("var_correction", ctypes.c_int32), ("pool_kernel", ctypes.c_int32),
                ("indicator_mode", ctypes.c_int32)]


_P = ctypes.c_void_p
_SIGNATURES = {
    "cake_version": (ctypes.c_int, []),
    "cake_last_error": (ctypes.c_char_p, []),
    "cake_workspace_bytes": (ctypes.c_int, [ctypes.POINTER(cake_shape), ctypes.POINTER(ctypes.c_size_t)]),
    "cake_window_scores": (ctypes.c_int, [ctypes.POINTER(cake_shape), ctypes.POINTER(cake_params), _P, _P,
                                          ctypes.POINTER(ctypes.c_int64), ctypes.POINTER(ctypes.c_int64), _P,
                                          _P, ctypes.c_size_t, _P]),
    "cake_window_scores_lse": (ctypes.c_int, [ctypes.POINTER(cake_shape), ctypes.POINTER(cake_params), _P, _P,
                                              ctypes.POINTER(ctypes.c_int64), ctypes.POINTER(ctypes.c_int64), _P, _P,
                                              _P, ctypes.c_size_t, _P]),
    "cake_scores_chunk_keys": (ctypes.c_int, [ctypes.POINTER(cake_shape), ctypes.POINTER(ctypes.c_int32)]),
    "cake_window_scores_segment": (ctypes.c_int, [ctypes.POINTER(cake_shape), ctypes.POINTER(cake_params), ctypes.c_int32,
                                                  ctypes.c_int32, ctypes.c_int32, _P, _P,
                                                  ctypes.POINTER(ctypes.c_int64), ctypes.POINTER(ctypes.c_int64),
                                                  _P, ctypes.c_size_t, _P]),
    "cake_window_scores_finish": (ctypes.c_int, [ctypes.POINTER(cake_shape), ctypes.POINTER(cake_params), ctypes.c_int32,
                                                 _P, _P, ctypes.c_size_t, _P]),
    "cake_layer_preference": (ctypes.c_int, [ctypes.POINTER(cake_shape), ctypes.POINTER(cake_params), _P,
                                             ctypes.c_size_t, _P, _P, _P]),
    "cake_keep_counts": (ctypes.c_int, [ctypes.POINTER(ctypes.c_int32), ctypes.POINTER(ctypes.c_int32), ctypes.c_int32,
                                        ctypes.c_int32, ctypes.POINTER(ctypes.c_int32)]),
    "cake_quantize_kv": (ctypes.c_int, [ctypes.POINTER(cake_shape), ctypes.c_int32, _P, _P, ctypes.POINTER(ctypes.c_int64),
                                        ctypes.POINTER(ctypes.c_int32), _P, _P, _P, _P, _P, _P, _P]),
    "cake_cascade_allocate": (ctypes.c_int, [ctypes.POINTER(ctypes.c_double), ctypes.c_int32, ctypes.c_int64,
                                             ctypes.c_int32, ctypes.c_int32, ctypes.POINTER(ctypes.c_int32)]),
    "cake_select_topk": (ctypes.c_int, [ctypes.POINTER(cake_shape), _P, ctypes.POINTER(ctypes.c_int32),
                                        ctypes.POINTER(ctypes.c_int32), _P, _P, ctypes.c_size_t, _P]),
    "cake_compact_kv": (ctypes.c_int, [ctypes.POINTER(cake_shape), _P, _P, ctypes.POINTER(ctypes.c_int64),
                                       ctypes.POINTER(ctypes.c_int32), ctypes.POINTER(ctypes.c_int32), _P, _P,
                                       _P, _P, _P, _P]),
    "cake_plan_bytes": (ctypes.c_int, [ctypes.POINTER(cake_shape), ctypes.POINTER(ctypes.c_size_t)]),
    "cake_plan_eviction": (ctypes.c_int, [ctypes.POINTER(cake_shape), _P, ctypes.c_int64, _P, _P, _P, _P, _P, _P,
                                          ctypes.c_size_t, _P, _P]),
    "cake_evict_planned": (ctypes.c_int, [ctypes.POINTER(cake_shape), _P, _P, _P, ctypes.POINTER(ctypes.c_int64),
                                          ctypes.POINTER(ctypes.c_uint8), _P, ctypes.c_size_t, _P]),
    "cake_plan_layout": (ctypes.c_int, [ctypes.POINTER(cake_shape), ctypes.POINTER(ctypes.c_size_t)]),
    "cake_decode_update": (ctypes.c_int, [ctypes.POINTER(cake_shape), ctypes.POINTER(cake_params), _P,
                                          ctypes.POINTER(ctypes.c_int64), _P, ctypes.POINTER(ctypes.c_int64),
                                          ctypes.POINTER(ctypes.c_int32), _P, _P, ctypes.c_size_t, _P]),
    "cake_decode_step_workspace_bytes": (ctypes.c_int, [ctypes.POINTER(cake_shape), ctypes.POINTER(ctypes.c_size_t)]),
    "cake_decode_step": (ctypes.c_int, [ctypes.POINTER(cake_shape), ctypes.POINTER(cake_params), _P,
                                        ctypes.POINTER(ctypes.c_int64), _P, _P, ctypes.POINTER(ctypes.c_int64), _P, _P,
                                        ctypes.POINTER(ctypes.c_int64), _P, _P, _P, ctypes.POINTER(ctypes.c_int32), _P,
                                        ctypes.c_size_t, _P]),
    "cake_decode_update_static": (ctypes.c_int, [ctypes.POINTER(cake_shape), ctypes.POINTER(cake_params), _P,
                                                 ctypes.POINTER(ctypes.c_int64), _P, ctypes.POINTER(ctypes.c_int64),
                                                 ctypes.POINTER(ctypes.c_int32), _P, _P]),
    "cake_profile_enable": (ctypes.c_int, [ctypes.c_int]),
    "cake_profile_read": (ctypes.c_int, [ctypes.POINTER(ctypes.c_float)]),
}

_lib = None


def load() -> ctypes.CDLL:
    """The loaded library.  Raises if libcake.so is absent: there is no fallback path."""
    global _lib
    if _lib is None:
        if not os.path.exists(LIB_PATH):
            raise ImportError(
                f"{LIB_PATH} is missing: build it with `python -m paper_2503_12491_amd.build` "
                "(hipcc, gfx950).  This package has no CPU or PyTorch fallback.")
        lib = ctypes.CDLL(LIB_PATH)
        for name, (res, args) in _SIGNATURES.items():
            fn = getattr(lib, name)
            fn.restype, fn.argtypes = res, args
        _lib = lib
    return _lib


class cake_pass(ctypes.Structure):
    """A one-shot pass described once (csrc/cake_pass.h)."""
    _fields_ = [("shape", cake_shape), ("params", cake_params)] + \
        [(n, _P) for n in ("q_win", "k", "v", "row_lse", "indicator")] + \
        [("q_strides", ctypes.c_int64 * 3), ("kv_strides", ctypes.c_int64 * 3), ("workspace", _P), ("workspace_bytes", ctypes.c_uint64),
         ("pref", _P), ("hv", _P), ("total_budget", ctypes.c_int64)] + \
        [(n, _P) for n in ("pool_idx", "pool_k", "pool_v", "pool_ind", "plan")] + \
        [("plan_bytes", ctypes.c_uint64), ("status", _P), ("mirror", _P)]


DECODE_LAYERS = 32


class cake_decode_plan(ctypes.Structure):
    """The buffers of an in-place decode step, described once (csrc/cake_pass.h)."""
    _fields_ = [("shape", cake_shape)] + \
        [(n, _P) for n in ("params", "k_slots", "v_slots", "indicator", "order", "state", "workspace")] + \
        [("workspace_bytes", ctypes.c_uint64), ("rank", ctypes.c_int64), ("slot_strides", ctypes.c_int64 * 3 * DECODE_LAYERS),
         ("cap", ctypes.c_int32 * DECODE_LAYERS), ("buffers", _P * 5 * DECODE_LAYERS)]


class cake_cascade(ctypes.Structure):
    """The buffers of a cascade chained on the device (csrc/cake_pass.h)."""
    _fields_ = [("shape", cake_shape), ("params", cake_params), ("max_layers", ctypes.c_int32), ("prefix_rows", ctypes.c_int32),
                ("total_budget", ctypes.c_int64), ("workspace", _P), ("workspace_bytes", ctypes.c_uint64)] + \
        [(n, _P) for n in ("pref", "hv", "status", "tables")] + [("plan", _P * 2), ("plan_bytes", ctypes.c_uint64),
         ("idx", _P), ("ind", _P * 2), ("slots", _P * 2)] + [(n, _P) for n in ("free_slots", "k_store", "v_store")]


class cake_session(ctypes.Structure):
    """A cascade whose allocation is the host's (csrc/cake_pass.h)."""
    _fields_ = [("shape", cake_shape), ("params", cake_params), ("max_layers", ctypes.c_int32), ("track_positions", ctypes.c_int32),
                ("total_budget", ctypes.c_int64), ("workspace", _P), ("workspace_bytes", ctypes.c_uint64)] + \
        [(n, _P) for n in ("mirror", "tables", "pref", "hv", "cur_len", "k", "v", "ind", "pos", "strides", "cap", "off_kv", "off_i",
                           "budgets")]


PASS_SCORES, PASS_EVICT = 1, 2
_host_module = None


def host():
    """The package's host module (csrc/host_module.cpp).  Raises if it has not been built."""
    global _host_module
    if _host_module is None:
        load()
        try:
            from . import _host as module
        except ImportError as e:
            raise ImportError(f"{e}: build it with `python -m paper_2503_12491_amd.build`") from e
        _host_module = module
    return _host_module


def mirror_layout(n_layers: int, batch: int) -> dict:
    """Byte offsets in a pass's pinned copy of the plan, and its size."""
    fn = load().cake_pass_mirror_layout
    fn.restype, fn.argtypes = None, [ctypes.c_int32, ctypes.c_int32, ctypes.POINTER(ctypes.c_uint64)]
    out = (ctypes.c_uint64 * 6)()
    fn(n_layers, batch, out)
    return dict(zip(("budgets", "keep", "status", "pref", "hv", "total"), [int(x) for x in out]))
