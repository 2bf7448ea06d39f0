"""Thin binding of the MDN C-ABI library (include/mdn.h).

Argument marshalling only: every step of the path runs in the HIP kernels of libmdn_hip.so.
PyTorch supplies device memory and the HIP stream.  There is no CPU fallback: a missing
library or a non-CUDA tensor raises.

The functions on tensors check their arguments, allocate outputs and call the library in the native module _mdn_torch
(csrc/mdn_torch.cpp: a decode step takes 4.4 us per call, with the same work in Python 12.9); size
queries, settings and the timing facility go through ctypes.
"""
from __future__ import annotations

import ctypes
import os

import torch

_HERE = os.path.dirname(os.path.abspath(__file__))
LIB_PATH = os.path.join(_HERE, "libmdn_hip.so")

MDN_DTYPE_BF16, MDN_DTYPE_F32 = 0, 1
MDN_WS_FWD, MDN_WS_BWD, MDN_WS_BWD_STATE_ADJOINTS = 0, 1, 2
MDN_WS_FWD_NO_STATES, MDN_WS_BWD_NO_STATES, MDN_WS_BWD_NO_STATE_ADJOINTS = 3, 4, 5 # packed batches only

EXPORTS = ("mdn_version", "mdn_strerror", "mdn_workspace_bytes", "mdn_saved_states_bytes",
           "mdn_saved_operands_bytes", "mdn_chunk_fwd", "mdn_chunk_fwd_noalloc",
           "mdn_chunk_bwd", "mdn_recurrent_step", "mdn_profile_begin", "mdn_profile_end", "mdn_profile_begin_sampled",
           "mdn_profile_launch_counts", "mdn_set_segments",
           "mdn_gates_fwd", "mdn_gates_bwd", "mdn_frontend_fwd", "mdn_frontend_bwd", "mdn_epilogue_fwd",
           "mdn_epilogue_bwd", "mdn_workspace_bytes_varlen", "mdn_chunk_fwd_varlen", "mdn_chunk_bwd_varlen")

KERNEL_NAMES = ("intra_fwd", "scan_fwd", "intra_bwd", "rebuild", "scan_bwd", "grad", "recurrent")


class MdnShape(ctypes.Structure):
    _fields_ = [("B", ctypes.c_int32), ("T", ctypes.c_int32), ("H", ctypes.c_int32), ("dk", ctypes.c_int32),
                ("dv", ctypes.c_int32), ("C", ctypes.c_int32), ("dtype", ctypes.c_int32), ("scale", ctypes.c_float)]


class MdnGateParams(ctypes.Structure):
    _fields_ = [("B", ctypes.c_int32), ("T", ctypes.c_int32), ("H", ctypes.c_int32), ("a_alpha", ctypes.c_void_p),
                ("b_alpha", ctypes.c_void_p), ("a_mu", ctypes.c_void_p), ("b_mu", ctypes.c_void_p),
                ("s", ctypes.c_float), ("tau", ctypes.c_float), ("mu_log_min", ctypes.c_float)]


class MdnError(RuntimeError):
    pass


_lib = None


def load_library():
    """dlopen libmdn_hip.so (built by __graft_entry__.build()) and declare the prototypes."""
    global _lib
    if _lib is not None:
        return _lib
    if not os.path.exists(LIB_PATH):
        raise MdnError(f"{LIB_PATH} is missing: run `python -c 'import __graft_entry__ as g; g.build()'` first")
    lib = ctypes.CDLL(LIB_PATH)
    vp, sp, fp = ctypes.c_void_p, ctypes.POINTER(MdnShape), ctypes.c_void_p
    lib.mdn_version.restype = ctypes.c_int
    lib.mdn_strerror.restype = ctypes.c_char_p
    lib.mdn_strerror.argtypes = [ctypes.c_int]
    lib.mdn_workspace_bytes.restype = ctypes.c_int
    lib.mdn_workspace_bytes.argtypes = [sp, ctypes.c_int, ctypes.POINTER(ctypes.c_size_t)]
    lib.mdn_saved_states_bytes.restype = ctypes.c_int
    lib.mdn_saved_states_bytes.argtypes = [sp, ctypes.POINTER(ctypes.c_size_t)]
    lib.mdn_saved_operands_bytes.restype = ctypes.c_int
    lib.mdn_saved_operands_bytes.argtypes = [sp, ctypes.POINTER(ctypes.c_size_t)]
    lib.mdn_chunk_fwd.restype = ctypes.c_int
    lib.mdn_chunk_fwd.argtypes = [sp] + [vp] * 3 + [fp] * 6 + [vp, fp, fp, vp, vp, vp, vp, ctypes.c_size_t, vp]
    lib.mdn_chunk_fwd_noalloc.restype = ctypes.c_int
    lib.mdn_chunk_fwd_noalloc.argtypes = [sp] + [vp] * 3 + [fp] * 6 + [vp, fp, fp, vp, vp]
    lib.mdn_chunk_bwd.restype = ctypes.c_int
    lib.mdn_chunk_bwd.argtypes = [sp] + [vp] * 3 + [fp] * 6 + [vp] * 4 + [fp] * 2 + [vp] * 3 + [fp] * 6 + \
        [vp, ctypes.c_size_t, vp]
    lib.mdn_recurrent_step.restype = ctypes.c_int
    lib.mdn_recurrent_step.argtypes = [sp] + [vp] * 3 + [fp] * 4 + [fp, fp, vp, vp]
    lib.mdn_profile_begin.restype = ctypes.c_int
    lib.mdn_profile_begin_sampled.restype = ctypes.c_int
    lib.mdn_profile_begin_sampled.argtypes = [ctypes.c_int]
    lib.mdn_profile_launch_counts.restype = ctypes.c_int
    lib.mdn_profile_launch_counts.argtypes = [ctypes.POINTER(ctypes.c_int), ctypes.c_int]
    lib.mdn_profile_end.restype = ctypes.c_int
    lib.mdn_profile_end.argtypes = [ctypes.POINTER(ctypes.c_float), ctypes.POINTER(ctypes.c_int), ctypes.c_int]
    lib.mdn_set_segments.restype = ctypes.c_int
    lib.mdn_set_segments.argtypes = [ctypes.c_int]
    gp = ctypes.POINTER(MdnGateParams)
    lib.mdn_gates_fwd.restype = ctypes.c_int
    lib.mdn_gates_fwd.argtypes = [gp] + [fp] * 8 + [vp]
    lib.mdn_gates_bwd.restype = ctypes.c_int
    lib.mdn_gates_bwd.argtypes = [gp] + [fp] * 13 + [vp]
    cf = ctypes.c_float
    ip = ctypes.POINTER(ctypes.c_int32)
    lib.mdn_workspace_bytes_varlen.restype = ctypes.c_int
    lib.mdn_workspace_bytes_varlen.argtypes = [sp, ip, ctypes.c_int32, ctypes.c_int, ctypes.POINTER(ctypes.c_size_t)]
    lib.mdn_chunk_fwd_varlen.restype = ctypes.c_int
    lib.mdn_chunk_fwd_varlen.argtypes = [sp, ip, ctypes.c_int32] + [vp] * 3 + [fp] * 6 + [vp, fp, fp, vp, vp, ctypes.c_size_t, vp]
    lib.mdn_chunk_bwd_varlen.restype = ctypes.c_int
    lib.mdn_chunk_bwd_varlen.argtypes = [sp, ip, ctypes.c_int32] + [vp] * 3 + [fp] * 6 + [vp, vp] + [fp] * 2 + [vp] * 3 + \
        [fp] * 6 + [vp, ctypes.c_size_t, vp]
    lib.mdn_frontend_fwd.restype = ctypes.c_int
    lib.mdn_frontend_fwd.argtypes = [sp, vp, vp, vp, fp, cf, vp, vp, vp, vp]
    lib.mdn_frontend_bwd.restype = ctypes.c_int
    lib.mdn_frontend_bwd.argtypes = [sp, vp, vp, vp, fp, cf] + [vp] * 6 + [fp, vp]
    lib.mdn_epilogue_fwd.restype = ctypes.c_int
    lib.mdn_epilogue_fwd.argtypes = [sp, vp, vp, fp, cf, vp, vp]
    lib.mdn_epilogue_bwd.restype = ctypes.c_int
    lib.mdn_epilogue_bwd.argtypes = [sp, vp, vp, fp, cf, vp, vp, vp, fp, vp]
    _lib = lib
    return lib


def _check(rc: int, what: str):
    if rc != 0:
        raise MdnError(f"{what}: {load_library().mdn_strerror(rc).decode()} (code {rc})")


_host = None


def _load_host():
    """Import the native module (built by __graft_entry__.build()) on top of the library."""
    global _host
    load_library()
    try:
        from . import _mdn_torch
    except ImportError as e:
        raise MdnError(f"the native binding module could not be loaded ({e}): run "
                       "`python -c 'import __graft_entry__ as g; g.build()'` first") from e
    _mdn_torch.set_error_types(MdnError, torch.OutOfMemoryError)
    _host = _mdn_torch
    return _host


def _dtype_code(t):
    if t.dtype == torch.bfloat16:
        return MDN_DTYPE_BF16
    if t.dtype == torch.float32:
        return MDN_DTYPE_F32
    raise MdnError("q/k/v must be bfloat16 or float32")


def make_shape(q, v, scale=None, C=64) -> MdnShape:
    B, T, H, dk = q.shape
    return MdnShape(B, T, H, dk, v.shape[-1], C, _dtype_code(q), float(dk ** -0.5 if scale is None else scale))


def workspace_bytes(shape: MdnShape, which: int) -> int:
    n = ctypes.c_size_t(0)
    _check(load_library().mdn_workspace_bytes(ctypes.byref(shape), which, ctypes.byref(n)), "mdn_workspace_bytes")
    return n.value


def saved_states_bytes(shape: MdnShape) -> int:
    n = ctypes.c_size_t(0)
    _check(load_library().mdn_saved_states_bytes(ctypes.byref(shape), ctypes.byref(n)), "mdn_saved_states_bytes")
    return n.value


def saved_operands_bytes(shape: MdnShape) -> int:
    n = ctypes.c_size_t(0)
    _check(load_library().mdn_saved_operands_bytes(ctypes.byref(shape), ctypes.byref(n)), "mdn_saved_operands_bytes")
    return n.value


def mdn_chunk_fwd(q, k, v, beta, alpha, mu, eta=None, S0=None, M0=None, scale=None, save_vt=False,
                  save_states=False, save_operands=False, output_final_state=True, workspace=None, out=None,
                  chunk_size=64):
    """Chunkwise forward.  Returns a dict: o, S, M (final states or None), vt, states, operands (or None), workspace;
    `out`: such a dict, whose tensors are reused."""
    return (_host or _load_host()).chunk_fwd(q, k, v, beta, alpha, mu, eta, S0, M0, scale, save_vt, save_states, save_operands,
                                             output_final_state, workspace, out, chunk_size)


def mdn_chunk_fwd_noalloc(q, k, v, beta, alpha, mu, out, eta=None, S0=None, M0=None, scale=None, chunk_size=64):
    """mdn_chunk_fwd through the entry point that allocates nothing: `out` holds the caller's o and, optionally, S, M
    and vt tensors (all of them preallocated; this function creates no tensor either).  Returns `out`."""
    return (_host or _load_host()).chunk_fwd_noalloc(q, k, v, beta, alpha, mu, out, eta, S0, M0, scale, chunk_size)


def mdn_chunk_bwd(q, k, v, beta, alpha, mu, vt, dO, eta=None, S0=None, M0=None, states=None, operands=None,
                  dS_final=None, dM_final=None, scale=None, want_deta=False, want_dstates=True, workspace=None, out=None,
                  chunk_size=64):
    """Chunkwise backward (chunk_size as in the forward call whose vt, states, operands it takes).  Returns a dict:
    dq, dk, dv, dbeta, dalpha, dmu, deta, dS0, dM0, workspace; `out`: such a dict, whose tensors are reused."""
    return (_host or _load_host()).chunk_bwd(q, k, v, beta, alpha, mu, vt, dO, eta, S0, M0, states, operands, dS_final, dM_final,
                                             scale, want_deta, want_dstates, workspace, out, chunk_size)


def mdn_recurrent_step(q, k, v, beta, alpha, mu, S, M, eta=None, scale=None, out=None):
    """Recurrent form over the T tokens given; S, M [B,H,dk,dv] fp32 are updated in place.  Returns o."""
    return (_host or _load_host()).recurrent_step(q, k, v, beta, alpha, mu, S, M, eta, scale, out)


def set_segments(k):
    """Force the number of sequence segments of mdn_chunk_fwd / mdn_chunk_bwd (0 = automatic); returns the old value."""
    return int(load_library().mdn_set_segments(int(k)))


def profile_begin(period=1):
    """Bracket every period-th launch of the library with an event pair (1 = every launch)."""
    _check(load_library().mdn_profile_begin_sampled(int(period)), "mdn_profile_begin_sampled")


def profile_end(with_launch_counts=False):
    """Per-kernel {name: (total_ms, bracketed launches)} since profile_begin(), with_launch_counts: (total_ms, bracketed
    launches, all launches); synchronises the recorded events."""
    n = len(KERNEL_NAMES)
    ms = (ctypes.c_float * n)()
    cnt = (ctypes.c_int * n)()
    every = (ctypes.c_int * n)()
    _check(load_library().mdn_profile_end(ms, cnt, n), "mdn_profile_end")
    _check(load_library().mdn_profile_launch_counts(every, n), "mdn_profile_launch_counts")
    if with_launch_counts:
        return {KERNEL_NAMES[i]: (float(ms[i]), int(cnt[i]), int(every[i])) for i in range(n)}
    return {KERNEL_NAMES[i]: (float(ms[i]), int(cnt[i])) for i in range(n)}


def mdn_gates_fwd(x_alpha, x_mu, x_beta, x_eta, a_alpha, b_alpha, a_mu, b_mu, s, tau, mu_log_min=-1.0):
    """Gate parameterisation: projections [B,T,H] fp32 -> dict(alpha, beta, mu, eta), each [B,T,H] fp32."""
    return (_host or _load_host()).gates_fwd(x_alpha, x_mu, x_beta, x_eta, a_alpha, b_alpha, a_mu, b_mu, s, tau, mu_log_min)


def mdn_gates_bwd(x_alpha, x_mu, x_beta, x_eta, a_alpha, b_alpha, a_mu, b_mu, s, tau, dalpha, dbeta, dmu, deta,
                  mu_log_min=-1.0, want_dparams=True):
    """Adjoint of mdn_gates_fwd: dict(dx_alpha, dx_mu, dx_beta, dx_eta [B,T,H]; dparams [4,H] = da_alpha, db_alpha,
    da_mu, db_mu, or None)."""
    return (_host or _load_host()).gates_bwd(x_alpha, x_mu, x_beta, x_eta, a_alpha, b_alpha, a_mu, b_mu, s, tau, dalpha, dbeta,
                                             dmu, deta, mu_log_min, want_dparams)


def mdn_frontend_fwd(x_q, x_k, x_v, d, eps=1e-6):
    """SiLU, output correction and L2 norms on the short-convolution outputs -> dict(q, k, v)."""
    return (_host or _load_host()).frontend_fwd(x_q, x_k, x_v, d, eps)


def mdn_frontend_bwd(x_q, x_k, x_v, d, dq, dk, dv, eps=1e-6, want_dd=True):
    """Adjoint of mdn_frontend_fwd: dict(dx_q, dx_k, dx_v, dd [H] or None)."""
    return (_host or _load_host()).frontend_bwd(x_q, x_k, x_v, d, dq, dk, dv, eps, want_dd)


def mdn_epilogue_fwd(o, g, w, eps=1e-6):
    """Head-wise RMS norm with weight w [dv] times sigmoid(g) -> y."""
    return (_host or _load_host()).epilogue_fwd(o, g, w, eps)


def mdn_epilogue_bwd(o, g, w, dy, eps=1e-6, want_dw=True):
    """Adjoint of mdn_epilogue_fwd: dict(do, dg, dw [dv] or None)."""
    return (_host or _load_host()).epilogue_bwd(o, g, w, dy, eps, want_dw)


def mdn_chunk_fwd_varlen(q, k, v, beta, alpha, mu, cu_seqlens, eta=None, S0=None, M0=None, scale=None, save_vt=False,
                         want_states=True):
    """Packed variable-length forward: q, k, v [1, T, H, d], gates [1, T, H], cu_seqlens a host sequence of n + 1
    offsets; states [n, H, dk, dv].  Returns dict(o, S, M, vt); S, M are None with want_states=False."""
    return (_host or _load_host()).chunk_fwd_varlen(q, k, v, beta, alpha, mu, cu_seqlens, eta, S0, M0, scale, save_vt, want_states)


def mdn_chunk_bwd_varlen(q, k, v, beta, alpha, mu, vt, dO, cu_seqlens, eta=None, S0=None, M0=None, dS_final=None,
                         dM_final=None, scale=None, want_deta=False, want_state_grads=True):
    """Packed variable-length backward.  Returns dict(dq, dk, dv, dbeta, dalpha, dmu, deta, dS0, dM0); dS0, dM0 are
    None with want_state_grads=False."""
    return (_host or _load_host()).chunk_bwd_varlen(q, k, v, beta, alpha, mu, vt, dO, cu_seqlens, eta, S0, M0, dS_final, dM_final,
                                                    scale, want_deta, want_state_grads)
