"""ctypes marshalling for include/fmbtf.h (same names as the C calls)."""
from __future__ import annotations

import ctypes as C
import os

import numpy as np

_PKG = os.path.dirname(os.path.abspath(__file__))
# FMBTF_LIB selects another build of the same library (the sanitizer build of
# the host code, for CPU checks)
_LIB_PATH = os.environ.get("FMBTF_LIB") or os.path.join(_PKG, "libfmbtf.so")

FM_OK, FM_EINVAL, FM_ESINGULAR, FM_ENOMEM, FM_EHIP, FM_ESTATE = 0, -1, -2, -3, -4, -5
FM_FP64, FM_FP32 = 64, 32
FM_DS_PER_PAIR, FM_DS_BROADCAST = 0, 1
FM_OUT_NODES, FM_OUT_RECEIVERS = 0, 1
FM_W_NODES, FM_W_RECEIVERS = 0, 1
FM_JT_PER_SOURCE, FM_JT_SUMMED = 0, 1

_ERRNAMES = {FM_EINVAL: "FM_EINVAL", FM_ESINGULAR: "FM_ESINGULAR", FM_ENOMEM: "FM_ENOMEM",
             FM_EHIP: "FM_EHIP", FM_ESTATE: "FM_ESTATE"}

SYMBOLS = (
    "fm_build_frozen_state", "fm_build_frozen_states", "fm_build_frozen_state_w", "fm_build_frozen_states_w",
    "fm_build_frozen_state_pt", "fm_build_frozen_states_pt", "fm_build_frozen_states_gpu",
    "fm_set_iterative_block_min", "fm_state_stats",
    "fm_state_export_operator", "fm_state_export_graph", "fm_state_free",
    "fm_batch_create", "fm_batch_set_stream", "fm_batch_tuning", "fm_batch_walk", "fm_batch_status", "fm_batch_split_info",
    "fm_apply_J", "fm_apply_J_static",
    "fm_apply_JT", "fm_apply_J_sweep", "fm_apply_JT_sweep", "fm_batch_free", "fm_last_error",
    "fm_lsqr_create", "fm_lsqr_start", "fm_lsqr_iterate", "fm_lsqr_capture", "fm_lsqr_replay",
    "fm_lsqr_buffers", "fm_lsqr_free", "fm_autotune",
    "fm_cgls_create", "fm_cgls_start", "fm_cgls_iterate", "fm_cgls_capture", "fm_cgls_replay",
    "fm_cgls_buffers", "fm_cgls_free",
    "fm_eikonal_create", "fm_eikonal_set_stream", "fm_eikonal_solve", "fm_eikonal_free",
    "fm_model_map_create", "fm_model_map_sizes", "fm_model_map_slowness", "fm_model_map_set_stream",
    "fm_model_map_apply", "fm_model_map_apply_T", "fm_model_map_free",
)


class FmError(RuntimeError):
    def __init__(self, code, msg):
        super().__init__(f"{_ERRNAMES.get(code, code)}: {msg}")
        self.code = code


class fm_grid(C.Structure):
    _fields_ = [("dim", C.c_int32), ("n1", C.c_int64), ("n2", C.c_int64), ("n3", C.c_int64),
                ("G", C.c_void_p), ("stencil", C.c_int32)]


class fm_stats(C.Structure):
    _fields_ = [("N", C.c_int64), ("E", C.c_int64), ("levels_fwd", C.c_int32),
                ("levels_rev", C.c_int32), ("n_scc", C.c_int32), ("largest_scc", C.c_int32),
                ("n_cyc", C.c_int64), ("sum_k2", C.c_int64), ("n_vio", C.c_int64),
                ("n_unr", C.c_int64), ("f_vio", C.c_double), ("f_cyc", C.c_double),
                ("f_unr", C.c_double), ("setup_seconds", C.c_double), ("state_bytes", C.c_int64),
                ("n_seed", C.c_int32), ("n_direct", C.c_int32), ("n_iter_blocks", C.c_int32),
                ("max_iter", C.c_int32), ("dense_k2", C.c_int64), ("iter_nnz", C.c_int64),
                ("block_residual", C.c_double)]


class fm_tuning(C.Structure):
    _fields_ = [("rhs_per_group", C.c_int32), ("threads", C.c_int32),
                ("min_lds_bytes", C.c_int32), ("xcd_aware", C.c_int32), ("unroll", C.c_int32),
                ("split", C.c_int32), ("balance", C.c_int32)]


class fm_walk(C.Structure):
    _fields_ = [("kernel", C.c_int32), ("threads", C.c_int32), ("unroll", C.c_int32),
                ("window", C.c_int32), ("side", C.c_int32)]


_lib = None


def lib_path() -> str:
    return _LIB_PATH


def load():
    """Load libfmbtf.so (raises if it is not built)."""
    global _lib
    if _lib is not None:
        return _lib
    if not os.path.exists(_LIB_PATH):
        raise ImportError(f"{_LIB_PATH} is not built: run __graft_entry__.build()")
    # torch brings its own HIP runtime; loading it first makes the library bind
    # to that same runtime instead of a second copy of it
    import torch  # noqa: F401
    lib = C.CDLL(_LIB_PATH)
    vp, i32, i64 = C.c_void_p, C.c_int32, C.c_int64
    sig = {
        "fm_build_frozen_state": (C.c_int, [vp, vp, vp, i64, vp, i32, vp]),
        "fm_build_frozen_states": (C.c_int, [vp, i32, vp, vp, vp, vp, i32, i32, vp]),
        "fm_build_frozen_state_w": (C.c_int, [vp, vp, vp, i64, vp, vp, i32, i32, vp]),
        "fm_build_frozen_states_w": (C.c_int, [vp, i32, vp, vp, vp, vp, vp, i32, i32, i32, vp]),
        "fm_build_frozen_state_pt": (C.c_int, [vp, vp, vp, vp, vp, C.c_double, vp, vp, i32, i32, vp]),
        "fm_build_frozen_states_pt": (C.c_int, [vp, vp, i32, vp, vp, vp, C.c_double, vp, vp, i32, i32, i32, vp]),
        "fm_set_iterative_block_min": (C.c_int, [i32]),
        "fm_build_frozen_states_gpu": (C.c_int, [vp, i32, vp, vp, vp, vp, vp, i32, i32, i32, vp, vp]),
        "fm_eikonal_create": (C.c_int, [i32, i64, i64, i64, vp, i32, vp, vp]),
        "fm_eikonal_set_stream": (C.c_int, [vp, vp]),
        "fm_eikonal_solve": (C.c_int, [vp, vp, i32, vp, C.c_double, i32, vp, vp]),
        "fm_eikonal_free": (None, [vp]),
        "fm_state_stats": (C.c_int, [vp, vp]),
        "fm_state_export_operator": (C.c_int, [vp, vp, vp, vp, vp]),
        "fm_state_export_graph": (C.c_int, [vp, vp, vp, vp]),
        "fm_state_free": (None, [vp]),
        "fm_batch_create": (C.c_int, [vp, i32, i32, i32, vp, vp, vp]),
        "fm_batch_set_stream": (C.c_int, [vp, vp]),
        "fm_autotune": (C.c_int, [vp, i32, i32, i32, vp, vp, i32, vp, i32, vp, i32, vp, i32, i32, C.c_char_p, vp,
                                  vp, vp, i32, vp]),
        "fm_batch_tuning": (C.c_int, [vp, vp]),
        "fm_batch_walk": (C.c_int, [vp, i32, vp]),
        "fm_batch_status": (C.c_int, [vp]),
        "fm_batch_split_info": (C.c_int, [vp, vp]),
        "fm_apply_J": (C.c_int, [vp, vp, i32, vp, i32]),
        "fm_apply_J_static": (C.c_int, [vp, i32, i32, i32, vp, vp, i32, vp, i32]),
        "fm_apply_JT": (C.c_int, [vp, vp, i32, vp, i32]),
        "fm_apply_J_sweep": (C.c_int, [vp, vp, i32, vp, i32, i32, vp]),
        "fm_apply_JT_sweep": (C.c_int, [vp, vp, vp, i32, i32, vp]),
        "fm_batch_free": (None, [vp]),
        "fm_lsqr_create": (C.c_int, [vp, vp]),
        "fm_lsqr_start": (C.c_int, [vp, vp]),
        "fm_lsqr_iterate": (C.c_int, [vp, i32]),
        "fm_lsqr_capture": (C.c_int, [vp, i32]),
        "fm_lsqr_replay": (C.c_int, [vp]),
        "fm_lsqr_buffers": (C.c_int, [vp, vp, vp, vp, vp]),
        "fm_lsqr_free": (None, [vp]),
        "fm_cgls_create": (C.c_int, [vp, i32, vp]),
        "fm_cgls_start": (C.c_int, [vp, vp]),
        "fm_cgls_iterate": (C.c_int, [vp, i32]),
        "fm_cgls_capture": (C.c_int, [vp, i32]),
        "fm_cgls_replay": (C.c_int, [vp]),
        "fm_cgls_buffers": (C.c_int, [vp, vp, vp, vp, vp]),
        "fm_cgls_free": (None, [vp]),
        "fm_last_error": (C.c_char_p, []),
        "fm_model_map_create": (C.c_int, [i32, i64, i64, i64, vp, vp, vp]),
        "fm_model_map_sizes": (C.c_int, [vp, vp, vp]),
        "fm_model_map_slowness": (C.c_int, [vp, vp]),
        "fm_model_map_set_stream": (C.c_int, [vp, vp]),
        "fm_model_map_apply": (C.c_int, [vp, i32, i32, vp, vp]),
        "fm_model_map_apply_T": (C.c_int, [vp, i32, i32, vp, vp]),
        "fm_model_map_free": (None, [vp]),
    }
    for name, (res, args) in sig.items():
        fn = getattr(lib, name)
        fn.restype = res
        fn.argtypes = args
    _lib = lib
    return lib


def exported_symbols():
    lib = load()
    return [s for s in SYMBOLS if hasattr(lib, s)]


def _check(rc):
    if rc != FM_OK:
        msg = load().fm_last_error().decode(errors="replace")
        raise FmError(rc, msg)


def _f64(a):
    return np.ascontiguousarray(a, dtype=np.float64)


def _i64(a):
    return np.ascontiguousarray(a, dtype=np.int64)


def _grid(dim, n1, n2, n3, G, stencil=6):
    g = fm_grid()
    g.dim, g.n1, g.n2, g.n3 = int(dim), int(n1), int(n2), int(n3)
    g.G = G.ctypes.data
    g.stencil = int(stencil)
    return g


class State:
    """One frozen source state (fm_state*)."""

    def __init__(self, ptr, N, dim, n, R):
        self._ptr = C.c_void_p(ptr)
        self.N = N
        self.dim = dim
        self.n = n
        self.R = R

    @property
    def ptr(self):
        return self._ptr

    def stats(self) -> dict:
        st = fm_stats()
        _check(load().fm_state_stats(self._ptr, C.byref(st)))
        return {k: getattr(st, k) for k, _ in fm_stats._fields_}

    def export_operator(self):
        """(rowptr [N+1], col [E], w [E], c [N]) of W in natural node order."""
        lib = load()
        rowptr = np.empty(self.N + 1, dtype=np.int64)
        _check(lib.fm_state_export_operator(self._ptr, rowptr.ctypes.data, None, None, None))
        E = int(rowptr[-1])
        col = np.empty(E, dtype=np.int32)
        w = np.empty(E, dtype=np.float64)
        c = np.empty(self.N, dtype=np.float64)
        _check(lib.fm_state_export_operator(self._ptr, rowptr.ctypes.data, col.ctypes.data,
                                            w.ctypes.data, c.ctypes.data))
        return rowptr, col, w, c

    def export_graph(self):
        comp = np.empty(self.N, dtype=np.int32)
        lf = np.empty(self.N, dtype=np.int32)
        lr = np.empty(self.N, dtype=np.int32)
        _check(load().fm_state_export_graph(self._ptr, comp.ctypes.data, lf.ctypes.data, lr.ctypes.data))
        return comp, lf, lr

    def free(self):
        if self._ptr and self._ptr.value:
            load().fm_state_free(self._ptr)
            self._ptr = C.c_void_p(None)

    def __del__(self):
        try:
            self.free()
        except Exception:
            pass


def build_frozen_state(dim, n1, n2, n3, G, T, s, src_node, rcv_nodes=(), rcv_weights=None, stencil=6) -> State:
    """fm_build_frozen_state with numpy host inputs.  With rcv_weights, the
    receivers interpolate: rcv_nodes and rcv_weights are [R][K] and receiver r
    samples sum_k rcv_weights[r][k] x[rcv_nodes[r][k]] (fm_build_frozen_state_w).
    stencil: 6 (faces) or 26 (cube), fm_grid.stencil."""
    lib = load()
    G, T, s = _f64(G), _f64(T), _f64(s)
    g = _grid(dim, n1, n2, n3, G, stencil)
    out = C.c_void_p()
    if rcv_weights is None:
        rcv = _i64(rcv_nodes)
        _check(lib.fm_build_frozen_state(C.byref(g), T.ctypes.data, s.ctypes.data, int(src_node),
                                         rcv.ctypes.data if rcv.size else None, int(rcv.size), C.byref(out)))
        R = int(rcv.size)
    else:
        rcv = np.ascontiguousarray(rcv_nodes, dtype=np.int64)
        w = np.ascontiguousarray(rcv_weights, dtype=np.float64)
        if rcv.ndim != 2 or w.shape != rcv.shape:
            raise ValueError("interpolating receivers need rcv_nodes and rcv_weights of one shape [R][K]")
        R, K = rcv.shape
        _check(lib.fm_build_frozen_state_w(C.byref(g), T.ctypes.data, s.ctypes.data, int(src_node),
                                           rcv.ctypes.data if rcv.size else None, w.ctypes.data if w.size else None,
                                           int(R), int(K), C.byref(out)))
    return State(out.value, int(n1) * int(n2) * int(n3), dim, (n1, n2, n3), int(R))


def build_frozen_states(dim, n1, n2, n3, G, T, s, src_nodes, rcv_nodes=None, nthreads=None, rcv_weights=None,
                        stencil=6):
    """fm_build_frozen_states: T [S][N]; rcv_nodes [R] (shared) or [S][R].
    With rcv_weights (fm_build_frozen_states_w): rcv_nodes and rcv_weights of
    one shape, [R][K] (shared) or [S][R][K], interpolating receivers.
    stencil: 6 (faces) or 26 (cube), fm_grid.stencil."""
    lib = load()
    G, T, s = _f64(G), _f64(T), _f64(s)
    src = _i64(src_nodes)
    S = int(src.shape[0])
    if nthreads is None:
        nthreads = min(16, os.cpu_count() or 1)
    g = _grid(dim, n1, n2, n3, G, stencil)
    outs = (C.c_void_p * S)()
    N = int(n1) * int(n2) * int(n3)
    if rcv_weights is not None:
        rcv = np.asarray(rcv_nodes, dtype=np.int64)
        w = np.asarray(rcv_weights, dtype=np.float64)
        if w.shape != rcv.shape or rcv.ndim not in (2, 3):
            raise ValueError("interpolating receivers need rcv_nodes and rcv_weights of one shape, "
                             "[R][K] or [S][R][K]")
        if rcv.ndim == 2:
            rcv = np.broadcast_to(rcv[None], (S,) + rcv.shape)
            w = np.broadcast_to(w[None], (S,) + w.shape)
        rcv, w = np.ascontiguousarray(rcv), np.ascontiguousarray(w)
        R, K = int(rcv.shape[1]), int(rcv.shape[2])
        _check(lib.fm_build_frozen_states_w(C.byref(g), S, T.ctypes.data, s.ctypes.data, src.ctypes.data,
                                            rcv.ctypes.data if rcv.size else None,
                                            w.ctypes.data if w.size else None, R, K, int(nthreads), outs))
        return [State(outs[a], N, dim, (n1, n2, n3), R) for a in range(S)]
    if rcv_nodes is None:
        rcv = np.zeros((S, 0), dtype=np.int64)
    else:
        rcv = np.asarray(rcv_nodes, dtype=np.int64)
        if rcv.ndim == 1:
            rcv = np.broadcast_to(rcv[None, :], (S, rcv.shape[0]))
        rcv = np.ascontiguousarray(rcv)
    _check(lib.fm_build_frozen_states(C.byref(g), S, T.ctypes.data, s.ctypes.data, src.ctypes.data,
                                      rcv.ctypes.data if rcv.size else None, int(rcv.shape[1]),
                                      int(nthreads), outs))
    return [State(outs[a], N, dim, (n1, n2, n3), int(rcv.shape[1])) for a in range(S)]


def build_frozen_states_gpu(dim, n1, n2, n3, G, T, s, src_nodes, rcv_nodes=None, rcv_weights=None, nthreads=None,
                            stream=None):
    """fm_build_frozen_states_gpu: T a device FP64 tensor [S][N] (the GPU setup
    pass computes the couplings); receivers as build_frozen_states."""
    import torch
    lib = load()
    G, s = _f64(G), _f64(s)
    src = _i64(src_nodes)
    S = int(src.shape[0])
    N = int(n1) * int(n2) * int(n3)
    if nthreads is None:
        nthreads = min(16, os.cpu_count() or 1)
    if stream is None:
        stream = torch.cuda.current_stream()
    g = _grid(dim, n1, n2, n3, G)
    outs = (C.c_void_p * S)()
    rcv, w = _receivers_pt(rcv_nodes, rcv_weights, S)
    R, K = int(rcv.shape[1]), int(rcv.shape[2])
    _check(lib.fm_build_frozen_states_gpu(C.byref(g), S, _dptr(T, torch.float64, (S, N), "T"), s.ctypes.data,
                                          src.ctypes.data, rcv.ctypes.data if rcv.size else None,
                                          w.ctypes.data if w is not None and w.size else None, R, K, int(nthreads),
                                          C.c_void_p(stream.cuda_stream), outs))
    return [State(outs[a], N, dim, (n1, n2, n3), R) for a in range(S)]


def set_iterative_block_min(k_min):
    """fm_set_iterative_block_min: states built from now on solve SCC blocks of
    at least k_min nodes by their Neumann series (0: default, < 0: never)."""
    _check(load().fm_set_iterative_block_min(int(k_min)))


def _receivers_pt(rcv_nodes, rcv_weights, S):
    """Receiver arrays [S][R][K] (nodes, weights or None) from [R], [R][K] or
    [S][R][K] inputs, shared across sources when given without S."""
    if rcv_nodes is None:
        return np.zeros((S, 0, 1), dtype=np.int64), None
    rcv = np.asarray(rcv_nodes, dtype=np.int64)
    if rcv_weights is None:
        if rcv.ndim == 1:
            rcv = np.broadcast_to(rcv[None], (S, rcv.shape[0]))
        if rcv.ndim != 2 or rcv.shape[0] != S:
            raise ValueError("receivers without weights are [R] (shared) or [S][R]")
        return np.ascontiguousarray(rcv.reshape(S, -1, 1)), None
    w = np.asarray(rcv_weights, dtype=np.float64)
    if w.shape != rcv.shape or rcv.ndim not in (2, 3):
        raise ValueError("interpolating receivers need rcv_nodes and rcv_weights of one shape, [R][K] or [S][R][K]")
    if rcv.ndim == 2:
        rcv = np.broadcast_to(rcv[None], (S,) + rcv.shape)
        w = np.broadcast_to(w[None], (S,) + w.shape)
    return np.ascontiguousarray(rcv), np.ascontiguousarray(w)


def build_frozen_states_pt(dim, n1, n2, n3, G, X, T, s, xi_src, seed_radius, rcv_nodes=None, rcv_weights=None,
                           nthreads=None, stencil=6):
    """fm_build_frozen_states_pt: off-grid point sources at logical
    coordinates xi_src [S][dim] with seed regions of max-norm radius
    seed_radius; X [N][dim] physical node coordinates, T [S][N] (straight-ray
    times over each seed region).  Receivers: [R] node selections or [R][K]
    nodes with rcv_weights [R][K] (shared by every source), or [S][R][K]."""
    lib = load()
    G, T, s, X = _f64(G), _f64(T), _f64(s), _f64(X)
    xi = np.ascontiguousarray(np.asarray(xi_src, dtype=np.float64).reshape(-1, dim))
    S = int(xi.shape[0])
    if T.size != S * int(n1) * int(n2) * int(n3):
        raise ValueError("T must be [S][N] with one row per source")
    if nthreads is None:
        nthreads = min(16, os.cpu_count() or 1)
    g = _grid(dim, n1, n2, n3, G, stencil)
    outs = (C.c_void_p * S)()
    N = int(n1) * int(n2) * int(n3)
    rcv, w = _receivers_pt(rcv_nodes, rcv_weights, S)
    R, K = int(rcv.shape[1]), int(rcv.shape[2])
    _check(lib.fm_build_frozen_states_pt(C.byref(g), X.ctypes.data, S, T.ctypes.data, s.ctypes.data, xi.ctypes.data,
                                         float(seed_radius), rcv.ctypes.data if rcv.size else None,
                                         w.ctypes.data if w is not None and w.size else None, R, K, int(nthreads),
                                         outs))
    return [State(outs[a], N, dim, (n1, n2, n3), R) for a in range(S)]


def _dptr(t, dtype, shape, what):
    import torch
    if not isinstance(t, torch.Tensor) or not t.is_cuda:
        raise ValueError(f"{what} must be a device tensor")
    if t.dtype != dtype:
        raise ValueError(f"{what} must be {dtype}, got {t.dtype}")
    if tuple(t.shape) != tuple(shape):
        raise ValueError(f"{what} must have shape {tuple(shape)}, got {tuple(t.shape)}")
    if not t.is_contiguous():
        raise ValueError(f"{what} must be contiguous")
    return C.c_void_p(t.data_ptr())


def default_tune_cache() -> str:
    """Where autotune keeps its results unless told otherwise: $FMBTF_TUNE_CACHE,
    else ~/.cache/fmbtf/autotune.txt."""
    path = os.environ.get("FMBTF_TUNE_CACHE")
    if path is not None:
        return path
    d = os.path.join(os.path.expanduser("~"), ".cache", "fmbtf")
    try:
        os.makedirs(d, exist_ok=True)
    except OSError:
        return ""
    return os.path.join(d, "autotune.txt")


def autotune(states, B, precision, ds, ds_mode, j_out, out_mode, w, w_mode, jt_out, jt_mode, reps=2, stream=None,
             cache=True):
    """fm_autotune on device tensors: returns (best tuning dict, [(tuning dict, ms per J + J^T pair), ...]).
    cache: True (default path), False (always search) or a file path; a cache
    hit returns the stored schedule and an empty candidate list."""
    import torch
    lib = load()
    states = list(states)
    S = len(states)
    arr = (C.c_void_p * S)(*[st.ptr.value for st in states])
    dt = torch.float64 if precision == FM_FP64 else torch.float32
    N, R = states[0].N, states[0].R
    B = int(B)
    ds_shape = (S, N, B) if ds_mode == FM_DS_PER_PAIR else (N, B)
    o_shape = (S, N, B) if out_mode == FM_OUT_NODES else (S, R, B)
    w_shape = (S, N, B) if w_mode == FM_W_NODES else (S, R, B)
    g_shape = (S, N, B) if jt_mode == FM_JT_PER_SOURCE else (N, B)
    if stream is None:
        stream = torch.cuda.current_stream()
    best = fm_tuning()
    n_max = 64
    cands = (fm_tuning * n_max)()
    ms = (C.c_float * n_max)()
    n = C.c_int32(0)
    path = default_tune_cache() if cache is True else (cache or "")
    _check(lib.fm_autotune(arr, S, B, int(precision), C.c_void_p(stream.cuda_stream),
                           _dptr(ds, dt, ds_shape, "ds"), int(ds_mode), _dptr(j_out, dt, o_shape, "j_out"),
                           int(out_mode), _dptr(w, dt, w_shape, "w"), int(w_mode), _dptr(jt_out, dt, g_shape, "jt_out"),
                           int(jt_mode), int(reps), path.encode(), C.byref(best), cands, ms, n_max, C.byref(n)))
    as_dict = lambda t: {k: getattr(t, k) for k, _ in fm_tuning._fields_}
    return as_dict(best), [(as_dict(cands[i]), float(ms[i])) for i in range(n.value)]


def apply_J_static(states, B, precision, ds, ds_mode, out, out_mode, stream=None):
    """fm_apply_J_static: J over resident states without a batch and without any
    device allocation (the library's fixed scratch array)."""
    import torch
    states = list(states)
    S, N, R = len(states), states[0].N, states[0].R
    B = int(B)
    dt = torch.float64 if precision == FM_FP64 else torch.float32
    arr = (C.c_void_p * S)(*[st.ptr.value for st in states])
    if stream is None:
        stream = torch.cuda.current_stream()
    ds_shape = (S, N, B) if ds_mode == FM_DS_PER_PAIR else (N, B)
    out_shape = (S, N, B) if out_mode == FM_OUT_NODES else (S, R, B)
    _check(load().fm_apply_J_static(arr, S, B, int(precision), C.c_void_p(stream.cuda_stream),
                                    _dptr(ds, dt, ds_shape, "ds"), int(ds_mode), _dptr(out, dt, out_shape, "out"),
                                    int(out_mode)))
    return out


class Batch:
    """fm_batch*: S states, B right-hand sides, preallocated scratch."""

    def __init__(self, states, B, precision=FM_FP64, tuning=None, stream=None):
        import torch
        lib = load()
        self.states = list(states)
        self.S = len(self.states)
        self.B = int(B)
        self.precision = precision
        self.N = self.states[0].N if self.states else 0     # no states: the library reports it
        self.dtype = torch.float64 if precision == FM_FP64 else torch.float32
        arr = (C.c_void_p * self.S)(*[st.ptr.value for st in self.states])
        tun = None
        if tuning is not None:
            tun = fm_tuning()
            for k, v in tuning.items():
                setattr(tun, k, int(v))
        if stream is None:
            stream = torch.cuda.current_stream()
        self._stream = stream
        out = C.c_void_p()
        _check(lib.fm_batch_create(arr, self.S, self.B, int(precision),
                                   C.byref(tun) if tun is not None else None,
                                   C.c_void_p(stream.cuda_stream), C.byref(out)))
        self._ptr = out
        self.R = self.states[0].R

    def tuning(self) -> dict:
        t = fm_tuning()
        _check(load().fm_batch_tuning(self._ptr, C.byref(t)))
        return {k: getattr(t, k) for k, _ in fm_tuning._fields_}

    def walk(self, transpose=False) -> dict:
        """The kernel that apply_J (or apply_JT) runs: "groups", "split" or "window"."""
        w = fm_walk()
        _check(load().fm_batch_walk(self._ptr, int(bool(transpose)), C.byref(w)))
        res = {k: getattr(w, k) for k, _ in fm_walk._fields_}
        res["kernel"] = ("groups", "split", "window")[w.kernel]
        return res

    def status(self):
        """Synchronise the batch stream; raises FmError if a node-split wait timed out."""
        _check(load().fm_batch_status(self._ptr))

    def split_info(self):
        """XCD bit mask per source of the last node-split apply."""
        m = np.zeros(self.S, dtype=np.int32)
        _check(load().fm_batch_split_info(self._ptr, m.ctypes.data))
        return m

    def set_stream(self, stream):
        _check(load().fm_batch_set_stream(self._ptr, C.c_void_p(stream.cuda_stream)))
        self._stream = stream

    def apply_J(self, ds, ds_mode, out, out_mode):
        S, N, B = self.S, self.N, self.B
        ds_shape = (S, N, B) if ds_mode == FM_DS_PER_PAIR else (N, B)
        out_shape = (S, N, B) if out_mode == FM_OUT_NODES else (S, self.R, B)
        _check(load().fm_apply_J(self._ptr, _dptr(ds, self.dtype, ds_shape, "ds"), int(ds_mode),
                                 _dptr(out, self.dtype, out_shape, "out"), int(out_mode)))
        return out

    def apply_JT(self, w, w_mode, out, out_mode):
        S, N, B = self.S, self.N, self.B
        w_shape = (S, N, B) if w_mode == FM_W_NODES else (S, self.R, B)
        out_shape = (S, N, B) if out_mode == FM_JT_PER_SOURCE else (N, B)
        _check(load().fm_apply_JT(self._ptr, _dptr(w, self.dtype, w_shape, "w"), int(w_mode),
                                  _dptr(out, self.dtype, out_shape, "out"), int(out_mode)))
        return out

    def _groups(self):
        return self.S * (self.B // self.tuning()["rhs_per_group"])

    def apply_J_sweep(self, ds, ds_mode, out, out_mode, max_cycles=10000, want_cycles=False):
        """Comparison baseline: J by directional Gauss-Seidel sweeping."""
        S, N, B = self.S, self.N, self.B
        ds_shape = (S, N, B) if ds_mode == FM_DS_PER_PAIR else (N, B)
        out_shape = (S, N, B) if out_mode == FM_OUT_NODES else (S, self.R, B)
        cyc = np.zeros(self._groups(), dtype=np.int32) if want_cycles else None
        _check(load().fm_apply_J_sweep(self._ptr, _dptr(ds, self.dtype, ds_shape, "ds"), int(ds_mode),
                                       _dptr(out, self.dtype, out_shape, "out"), int(out_mode),
                                       int(max_cycles), cyc.ctypes.data if cyc is not None else None))
        return cyc

    def apply_JT_sweep(self, w, out, out_mode, max_cycles=10000, want_cycles=False):
        """Comparison baseline: J^T (nodal input) by directional Gauss-Seidel sweeping."""
        S, N, B = self.S, self.N, self.B
        out_shape = (S, N, B) if out_mode == FM_JT_PER_SOURCE else (N, B)
        cyc = np.zeros(self._groups(), dtype=np.int32) if want_cycles else None
        _check(load().fm_apply_JT_sweep(self._ptr, _dptr(w, self.dtype, (S, N, B), "w"),
                                        _dptr(out, self.dtype, out_shape, "out"), int(out_mode),
                                        int(max_cycles), cyc.ctypes.data if cyc is not None else None))
        return cyc

    def free(self):
        if getattr(self, "_ptr", None) is not None and self._ptr.value:
            load().fm_batch_free(self._ptr)
            self._ptr = C.c_void_p(None)

    def __del__(self):
        try:
            self.free()
        except Exception:
            pass


class ModelMap:
    """fm_model_map*: cell velocities -> nodal slowness, linearised (M of
    Section 4.4, eq. (source-jacobian)) and its transpose, on the GPU."""

    def __init__(self, dim, n1, n2, n3, v_cell, stream=None):
        import torch
        lib = load()
        v = _f64(v_cell)
        if stream is None:
            stream = torch.cuda.current_stream()
        out = C.c_void_p()
        _check(lib.fm_model_map_create(int(dim), int(n1), int(n2), int(n3), v.ctypes.data,
                                       C.c_void_p(stream.cuda_stream), C.byref(out)))
        self._ptr = out
        nn, nc = C.c_int64(), C.c_int64()
        _check(lib.fm_model_map_sizes(out, C.byref(nn), C.byref(nc)))
        self.N, self.n_cells = int(nn.value), int(nc.value)

    def slowness(self) -> np.ndarray:
        s = np.empty(self.N, dtype=np.float64)
        _check(load().fm_model_map_slowness(self._ptr, s.ctypes.data))
        return s

    def set_stream(self, stream):
        _check(load().fm_model_map_set_stream(self._ptr, C.c_void_p(stream.cuda_stream)))

    def _prec(self, t):
        import torch
        return FM_FP64 if t.dtype == torch.float64 else FM_FP32

    def apply(self, dv, ds):
        """ds [N][B] = M dv [n_cells][B] (device tensors of one dtype)."""
        B = int(dv.shape[1])
        _check(load().fm_model_map_apply(self._ptr, B, self._prec(dv), _dptr(dv, dv.dtype, (self.n_cells, B), "dv"),
                                         _dptr(ds, dv.dtype, (self.N, B), "ds")))

    def apply_T(self, g, out):
        """out [n_cells][B] = M^T g [N][B]."""
        B = int(g.shape[1])
        _check(load().fm_model_map_apply_T(self._ptr, B, self._prec(g), _dptr(g, g.dtype, (self.N, B), "g"),
                                           _dptr(out, g.dtype, (self.n_cells, B), "out")))

    def free(self):
        if self._ptr and self._ptr.value:
            load().fm_model_map_free(self._ptr)
            self._ptr = C.c_void_p(None)

    def __del__(self):
        try:
            self.free()
        except Exception:
            pass


class Eikonal:
    """fm_eikonal*: first-arrival traveltimes for many sources on the GPU
    (the monotone semi-Lagrangian update; Section 2.1's state)."""

    def __init__(self, dim, n1, n2, n3, X, max_sources, stream=None):
        import torch
        lib = load()
        X = _f64(X)
        if stream is None:
            stream = torch.cuda.current_stream()
        self._stream = stream
        out = C.c_void_p()
        _check(lib.fm_eikonal_create(int(dim), int(n1), int(n2), int(n3), X.ctypes.data, int(max_sources),
                                     C.c_void_p(stream.cuda_stream), C.byref(out)))
        self._ptr = out
        self.dim, self.N, self.max_sources = int(dim), int(n1) * int(n2) * int(n3), int(max_sources)

    def solve(self, s, xi_src, seed_radius, out, max_iter=100000):
        """out [S][N] (device FP64) <- traveltimes for slowness s [N] (device
        FP64) and sources at logical coordinates xi_src [S][dim] (host);
        returns the number of Jacobi iterations."""
        import torch
        xi = np.ascontiguousarray(np.asarray(xi_src, dtype=np.float64).reshape(-1, self.dim))
        S = int(xi.shape[0])
        it = C.c_int32()
        _check(load().fm_eikonal_solve(self._ptr, _dptr(s, torch.float64, (self.N,), "s"), S, xi.ctypes.data,
                                       float(seed_radius), int(max_iter),
                                       _dptr(out, torch.float64, (S, self.N), "T"), C.byref(it)))
        return int(it.value)

    def free(self):
        if self._ptr and self._ptr.value:
            load().fm_eikonal_free(self._ptr)
            self._ptr = C.c_void_p(None)

    def __del__(self):
        try:
            self.free()
        except Exception:
            pass


class Lsqr:
    """fm_lsqr*: LSQR over the paired actions of a batch (device-resident)."""

    def __init__(self, batch: Batch):
        self.batch = batch
        out = C.c_void_p()
        _check(load().fm_lsqr_create(batch._ptr, C.byref(out)))
        self._ptr = out
        ptrs = [C.c_void_p() for _ in range(4)]
        _check(load().fm_lsqr_buffers(self._ptr, *[C.byref(p) for p in ptrs]))
        self._x, self._u, self._v, self._scal = (p.value for p in ptrs)

    def start(self, d):
        b = self.batch
        _check(load().fm_lsqr_start(self._ptr, _dptr(d, b.dtype, (b.S, b.R, b.B), "d")))

    def iterate(self, n):
        _check(load().fm_lsqr_iterate(self._ptr, int(n)))

    def capture(self, n):
        _check(load().fm_lsqr_capture(self._ptr, int(n)))

    def replay(self):
        _check(load().fm_lsqr_replay(self._ptr))

    def x(self):
        """A device copy of the current solution [N][B]."""
        return _device_copy(self._x, (self.batch.N, self.batch.B), self.batch.dtype)

    def scalars(self):
        """Per-column scalars [8][B]: alpha, beta, rhobar, phibar, rho, phi, theta, 1/norm."""
        import torch
        return _device_copy(self._scal, (8, self.batch.B), torch.float64)

    def free(self):
        if getattr(self, "_ptr", None) is not None and self._ptr.value:
            load().fm_lsqr_free(self._ptr)
            self._ptr = C.c_void_p(None)

    def __del__(self):
        try:
            self.free()
        except Exception:
            pass


class Cgls:
    """fm_cgls*: CGLS over the paired actions of a batch (device-resident)."""

    def __init__(self, batch: Batch, max_iter: int = 100):
        self.batch = batch
        self.max_iter = int(max_iter)
        out = C.c_void_p()
        _check(load().fm_cgls_create(batch._ptr, self.max_iter, C.byref(out)))
        self._ptr = out
        ptrs = [C.c_void_p() for _ in range(4)]
        _check(load().fm_cgls_buffers(self._ptr, *[C.byref(p) for p in ptrs]))
        self._x, self._r, self._scal, self._hist = (p.value for p in ptrs)

    def start(self, d):
        b = self.batch
        _check(load().fm_cgls_start(self._ptr, _dptr(d, b.dtype, (b.S, b.R, b.B), "d")))

    def iterate(self, n):
        _check(load().fm_cgls_iterate(self._ptr, int(n)))

    def capture(self, n):
        _check(load().fm_cgls_capture(self._ptr, int(n)))

    def replay(self):
        _check(load().fm_cgls_replay(self._ptr))

    def x(self):
        """A device copy of the current solution [N][B]."""
        return _device_copy(self._x, (self.batch.N, self.batch.B), self.batch.dtype)

    def residual(self):
        """A device copy of the current data residual r = d - J x [S][R][B]."""
        b = self.batch
        return _device_copy(self._r, (b.S, b.R, b.B), b.dtype)

    def scalars(self):
        """Per-column scalars [6][B]: gamma, ||q||^2, alpha, gamma', beta, ||r||^2."""
        import torch
        return _device_copy(self._scal, (6, self.batch.B), torch.float64)

    def history(self):
        """||r||^2 per column after start and after each iteration: [max_iter + 1][B]."""
        import torch
        return _device_copy(self._hist, (self.max_iter + 1, self.batch.B), torch.float64)

    def free(self):
        if getattr(self, "_ptr", None) is not None and self._ptr.value:
            load().fm_cgls_free(self._ptr)
            self._ptr = C.c_void_p(None)

    def __del__(self):
        try:
            self.free()
        except Exception:
            pass


def _device_copy(ptr, shape, dtype):
    """Copy a library-owned device buffer into a new torch tensor."""
    import torch
    out = torch.empty(shape, dtype=dtype, device="cuda")
    nbytes = out.numel() * out.element_size()
    torch.cuda.synchronize()
    hip = C.CDLL("libamdhip64.so")
    hip.hipMemcpy.restype = C.c_int
    hip.hipMemcpy.argtypes = [C.c_void_p, C.c_void_p, C.c_size_t, C.c_int]
    rc = hip.hipMemcpy(C.c_void_p(out.data_ptr()), C.c_void_p(ptr), nbytes, 3)   # device to device
    if rc != 0:
        raise FmError(FM_EHIP, f"hipMemcpy failed: {rc}")
    return out
