"""Binding of libcorey.so: argument marshalling only.

Functions carry the names of the C entry points (include/corey.h).  Device buffers are torch tensors
(torch is used for GPU memory and streams, nothing else); every step of the path runs in the library's
HIP kernels.  Calls on tensors go through the extension `_native` (csrc/corey_torch.cpp), which checks and converts their
arguments in native code; the host functions and the raw C ABI (`lib()`) through ctypes.  There is no fallback: if the
library or the extension is missing or fails to load, calls raise.
"""
from __future__ import annotations

import ctypes
import os

import torch

_HERE = os.path.dirname(os.path.abspath(__file__))
LIB_PATH = os.environ.get("COREY_LIB") or os.path.join(_HERE, "libcorey.so")   # COREY_LIB: another build of the same library

COREY_F32, COREY_BF16, COREY_F16 = 0, 1, 2
STATUS = {0: "COREY_OK", 1: "COREY_EINVAL", 2: "COREY_ENULL", 3: "COREY_ESHAPE", 4: "COREY_ENONFINITE",
          5: "COREY_EUNSUPPORTED", 6: "COREY_EHIP", 7: "COREY_EWORKSPACE"}
EXPORTS = ("corey_entropy_hist", "corey_entropy_hist_static", "corey_entropy_hist_workspace", "corey_pattern_table_workspace",
           "corey_entropy_hist_onesweep", "corey_entropy_hist_from_table", "corey_policy_default", "corey_select_chunk",
           "corey_select_chunk_device", "corey_route_device", "corey_route_device_deferred", "selective_scan_fwd_routed", "corey_ema_update", "causal_conv1d_silu_fwd", "selective_state_update",
           "selective_scan_fwd", "selective_scan_fwd_workspace", "selective_scan_fwd_plan", "selective_scan_fwd_plan_steps", "selective_scan_fwd_plan_split", "corey_last_error", "corey_version")


class CoreyError(RuntimeError):
    def __init__(self, code: int, msg: str):
        super().__init__(f"{STATUS.get(code, code)}: {msg}")
        self.code = code


class Policy(ctypes.Structure):
    """corey_policy"""
    _fields_ = [("mode", ctypes.c_int32), ("c_min", ctypes.c_int32), ("c_max", ctypes.c_int32),
                ("h_ref_scale", ctypes.c_double), ("short_len", ctypes.c_int32), ("short_chunk", ctypes.c_int32),
                ("long_chunk", ctypes.c_int32), ("static_chunk", ctypes.c_int32), ("safe_chunk", ctypes.c_int32),
                ("guard_buckets", ctypes.c_int32)]


class DeferredRoute(ctypes.Structure):
    """corey_deferred_route: opaque, filled by corey_route_device_deferred, consumed by selective_scan_fwd_routed"""
    _fields_ = [("opaque", ctypes.c_uint64 * 40)]


_lib = None


def lib() -> ctypes.CDLL:
    """Load libcorey.so (built in-tree by build.py); raises if it is not there."""
    global _lib
    if _lib is None:
        if not os.path.exists(LIB_PATH):
            raise ImportError(f"{LIB_PATH} is missing: run `python -c 'import __graft_entry__ as g; g.build()'`")
        L = ctypes.CDLL(LIB_PATH)
        i64, i32, vp, dbl = ctypes.c_int64, ctypes.c_int32, ctypes.c_void_p, ctypes.c_double
        L.corey_entropy_hist.restype = ctypes.c_int
        L.corey_entropy_hist.argtypes = [vp, ctypes.c_int, i64, i64, i64, vp, i32, dbl, i64, i64, vp, vp, vp, vp, vp, vp,
                                         ctypes.c_size_t, vp]
        L.corey_entropy_hist_static.restype = ctypes.c_int
        L.corey_entropy_hist_static.argtypes = [vp, ctypes.c_int, i64, i64, i64, vp, i32, dbl, i64, i64, vp, vp, vp, vp, vp, vp]
        L.corey_pattern_table_workspace.restype = ctypes.c_size_t
        L.corey_pattern_table_workspace.argtypes = []
        L.corey_entropy_hist_onesweep.restype = ctypes.c_int
        L.corey_entropy_hist_onesweep.argtypes = [vp, ctypes.c_int, i64, i64, i64, i32, dbl, ctypes.POINTER(Policy), vp, vp, vp, vp, vp, vp,
                                                  ctypes.c_size_t, vp]
        L.corey_entropy_hist_from_table.restype = ctypes.c_int
        L.corey_entropy_hist_from_table.argtypes = [ctypes.c_int, i64, i32, dbl, ctypes.POINTER(Policy), vp, vp, vp, vp, vp, vp,
                                                    ctypes.c_size_t, vp]
        L.selective_state_update.restype = ctypes.c_int
        L.selective_state_update.argtypes = [vp, vp, vp, vp, vp, vp, vp, vp, vp, i32, vp, ctypes.c_int, i64, i64, i64, vp]
        L.causal_conv1d_silu_fwd.restype = ctypes.c_int
        L.causal_conv1d_silu_fwd.argtypes = [vp, vp, vp, vp, vp, vp, vp, vp, ctypes.c_size_t, ctypes.c_int, i64, i64, i64, i32, vp]
        L.corey_route_device.restype = ctypes.c_int
        L.corey_route_device.argtypes = [vp, ctypes.c_int, i64, i64, i64, vp, i32, dbl, i64, i64, ctypes.POINTER(Policy), dbl, vp, vp,
                                         vp, vp, vp, vp, vp, vp, vp, ctypes.c_size_t, vp]
        L.corey_route_device_deferred.restype = ctypes.c_int
        L.corey_route_device_deferred.argtypes = [vp, ctypes.c_int, i64, i64, i64, vp, i32, dbl, i64, i64, ctypes.POINTER(Policy), vp,
                                                  vp, vp, vp, vp, vp, vp, vp, ctypes.c_size_t, ctypes.POINTER(DeferredRoute), vp]
        L.selective_scan_fwd_routed.restype = ctypes.c_int
        L.selective_scan_fwd_routed.argtypes = [vp, vp, vp, vp, vp, vp, vp, vp, ctypes.c_int, vp, vp, i32, ctypes.POINTER(DeferredRoute),
                                                vp, vp, ctypes.c_int, i64, i64, i64, i64, ctypes.c_uint32, vp, ctypes.c_size_t, vp]
        L.corey_ema_update.restype = ctypes.c_int
        L.corey_ema_update.argtypes = [dbl, ctypes.POINTER(dbl), dbl]
        L.corey_entropy_hist_workspace.restype = ctypes.c_size_t
        L.corey_entropy_hist_workspace.argtypes = [i64, i32]
        L.corey_policy_default.restype = ctypes.c_int
        L.corey_policy_default.argtypes = [ctypes.POINTER(Policy)]
        L.corey_select_chunk.restype = ctypes.c_int
        L.corey_select_chunk.argtypes = [dbl, i64, ctypes.POINTER(Policy), ctypes.POINTER(i32)]
        L.corey_select_chunk_device.restype = ctypes.c_int
        L.corey_select_chunk_device.argtypes = [vp, vp, i64, i32, ctypes.POINTER(Policy), vp, vp]
        L.selective_scan_fwd.restype = ctypes.c_int
        L.selective_scan_fwd.argtypes = [vp, vp, vp, vp, vp, vp, vp, vp, ctypes.c_int, vp, vp, i32, vp, vp, vp,
                                         ctypes.c_int, i64, i64, i64, i64, ctypes.c_uint32, vp, ctypes.c_size_t, vp]
        L.selective_scan_fwd_plan.restype = ctypes.c_int64
        L.selective_scan_fwd_plan.argtypes = [i64, i64, i64, i32]
        L.selective_scan_fwd_plan_steps.restype = i32
        L.selective_scan_fwd_plan_steps.argtypes = [i64, i64, i64, i32]
        L.selective_scan_fwd_plan_split.restype = i32
        L.selective_scan_fwd_plan_split.argtypes = [i64, i64, i64, i32]
        L.selective_scan_fwd_workspace.restype = ctypes.c_size_t
        L.selective_scan_fwd_workspace.argtypes = [i64, i64, i64]
        L.corey_last_error.restype = ctypes.c_char_p
        L.corey_version.restype = ctypes.c_char_p
        _lib = L
    return _lib


_ext = None


def _native():
    """The torch extension, on the library that lib() loads; raises if either is not there."""
    global _ext
    if _ext is None:
        lib()
        from . import _native as ext      # built in-tree by build.py
        ext.attach(LIB_PATH, CoreyError, DeferredRoute)
        _ext = ext
    return _ext


def _check(code: int):
    if code != 0:
        raise CoreyError(code, lib().corey_last_error().decode())


def _ptr(t):
    return None if t is None else ctypes.c_void_p(t.data_ptr())


def _dtype_code(t: torch.Tensor) -> int:
    if t.dtype == torch.float32:
        return COREY_F32
    if t.dtype == torch.bfloat16:
        return COREY_BF16
    if t.dtype == torch.float16:
        return COREY_F16
    raise TypeError(f"unsupported storage type {t.dtype}")


def _stream():
    return ctypes.c_void_p(torch.cuda.current_stream().cuda_stream)


def policy_default() -> Policy:
    p = Policy()
    _check(lib().corey_policy_default(ctypes.byref(p)))
    return p


def corey_version() -> str:
    return lib().corey_version().decode()


def corey_entropy_hist_workspace(B: int, K: int) -> int:
    return int(lib().corey_entropy_hist_workspace(B, K))


def selective_state_update(state: torch.Tensor, x: torch.Tensor, delta: torch.Tensor, A: torch.Tensor, Bt: torch.Tensor,
                           Ct: torch.Tensor, Dv: torch.Tensor | None = None, z: torch.Tensor | None = None,
                           delta_bias: torch.Tensor | None = None, delta_softplus: bool = True, y: torch.Tensor | None = None):
    """One decode step: state float32 [B, D, N] is updated in place; x, delta, z [B, D]; Bt, Ct [B, N]; returns y [B, D]."""
    return (_ext or _native()).selective_state_update(state, x, delta, A, Bt, Ct, Dv, z, delta_bias, delta_softplus, y)


HANDOFF_BYTES = 1024 * 16 + 16 * 4096 * 4      # COREY_HANDOFF_BYTES: partial ranges + partial histograms
RANGE_PARTS_BYTES = HANDOFF_BYTES
CHUNK_SLOTS = 12                   # COREY_CHUNK_SLOTS


def causal_conv1d_silu_fwd(x: torch.Tensor, weight: torch.Tensor, bias: torch.Tensor | None = None,
                           state_in: torch.Tensor | None = None, u: torch.Tensor | None = None, want_state: bool = False,
                           range_parts: torch.Tensor | None = None, pattern_table: torch.Tensor | None = None):
    """x [B, D, L] GPU tensor, weight float32 [D, W], bias float32 [D].  Returns (u, state_out or None, range_parts):
    range_parts (uint8 GPU tensor of HANDOFF_BYTES, allocated here if omitted) can be handed to
    corey_entropy_hist / corey_route_device on this u, which then skip their range sweep.  pattern_table: uint8 GPU
    tensor of corey_pattern_table_workspace() bytes; the kernel then also fills the bit-pattern table of u for
    corey_entropy_hist_from_table."""
    return (_ext or _native()).causal_conv1d_silu_fwd(x, weight, bias, state_in, u, want_state, range_parts, pattern_table)


def corey_entropy_hist(x: torch.Tensor, K: int, eps: float = 1e-8, stride: int = 1, seqlens: torch.Tensor | None = None,
                       out: dict | None = None, workspace: torch.Tensor | None = None, block: int = 1,
                       range_parts: torch.Tensor | None = None):
    """x: [B, D, L] GPU tensor (float32 or bfloat16).  Returns dict(counts, H, r, range) of GPU tensors;
    nothing is copied to the host and the call does not synchronise."""
    return (_ext or _native()).corey_entropy_hist(x, K, eps, stride, seqlens, out, workspace, block, range_parts)


def corey_pattern_table_workspace() -> int:
    return int(lib().corey_pattern_table_workspace())


def corey_entropy_hist_onesweep(x: torch.Tensor, K: int, eps: float = 1e-8, policy: Policy | None = None, out: dict | None = None,
                                table_ws: torch.Tensor | None = None):
    """The statistic of a bfloat16 / float16 tensor from one pass over it (bit-pattern table).  Returns the dict of
    corey_entropy_hist (plus `chunks` when a policy is given, as corey_route_device) and `table_ws`."""
    return (_ext or _native()).corey_entropy_hist_onesweep(x, K, eps, policy, out, table_ws)


def corey_entropy_hist_from_table(table_ws: torch.Tensor, dtype: torch.dtype, L: int, K: int, eps: float = 1e-8,
                                  policy: Policy | None = None, out: dict | None = None):
    """The statistic of the tensor whose producer (causal_conv1d_silu_fwd with pattern_table=table_ws) filled the table."""
    code = {torch.bfloat16: COREY_BF16, torch.float16: COREY_F16, torch.float32: COREY_F32}[dtype]
    return (_ext or _native()).corey_entropy_hist_from_table(table_ws, code, L, K, eps, policy, out)


STATIC_SCRATCH_BYTES = 1 << 20     # COREY_STATIC_SCRATCH_BYTES


def corey_entropy_hist_static(x: torch.Tensor, K: int, out: dict, eps: float = 1e-8, stride: int = 1,
                              seqlens: torch.Tensor | None = None, block: int = 1, range_parts: torch.Tensor | None = None):
    """corey_entropy_hist on the library's built-in scratch buffer: nothing is allocated, here or in the library, so
    `out` (dict(counts, H, r[, range]) of GPU tensors, as corey_entropy_hist returns) must be given."""
    return (_ext or _native()).corey_entropy_hist_static(x, K, out, eps, stride, seqlens, block, range_parts)


def corey_ema_update(lam: float, state: float, H: float) -> float:
    """One step of the entropy EMA on the host; state = NaN means no estimate yet.  Returns the new state."""
    st = ctypes.c_double(state)
    _check(lib().corey_ema_update(float(lam), ctypes.byref(st), float(H)))
    return st.value


def corey_route_device(x: torch.Tensor, K: int, policy: Policy | None = None, eps: float = 1e-8, stride: int = 1, block: int = 1,
                       seqlens: torch.Tensor | None = None, out: dict | None = None, workspace: torch.Tensor | None = None,
                       ema_lambda: float = 0.0, ema_state: torch.Tensor | None = None, chunk_calls: torch.Tensor | None = None,
                       range_parts: torch.Tensor | None = None):
    """corey_entropy_hist and the chunk rule in one call.  Returns the dict of corey_entropy_hist plus `chunks`
    (int32 GPU tensor [nh], directly usable as `chunks_dev` of selective_scan_fwd); no synchronisation.
    ema_state: float64 GPU tensor [nh] (NaN = no estimate yet), updated in place; chunk_calls: int32 GPU tensor
    [COREY_CHUNK_SLOTS] of counters the caller clears."""
    return (_ext or _native()).corey_route_device(x, K, policy, eps, stride, block, seqlens, out, workspace, chunk_calls, range_parts,
                                                  ema_lambda, ema_state)


def corey_route_device_deferred(x: torch.Tensor, K: int, policy: Policy | None = None, eps: float = 1e-8, stride: int = 1, block: int = 1,
                                seqlens: torch.Tensor | None = None, out: dict | None = None, workspace: torch.Tensor | None = None,
                                chunk_calls: torch.Tensor | None = None, range_parts: torch.Tensor | None = None):
    """The sweeps of corey_route_device without its reduction: returns the same dict (its tensors are written by the
    selective_scan_fwd_routed call that follows) with `route`, the ticket that call takes."""
    return (_ext or _native()).corey_route_device_deferred(x, K, policy, eps, stride, block, seqlens, out, workspace, chunk_calls,
                                                           range_parts)


def corey_select_chunk(r: float, L: int, policy: Policy | None = None) -> int:
    p = policy if policy is not None else policy_default()
    c = ctypes.c_int32(0)
    _check(lib().corey_select_chunk(float(r), int(L), ctypes.byref(p), ctypes.byref(c)))
    return c.value


def corey_select_chunk_device(r_dev: torch.Tensor, L: int, policy: Policy | None = None, seqlens: torch.Tensor | None = None,
                              out: torch.Tensor | None = None) -> torch.Tensor:
    """r_dev: float64 GPU tensor [nh].  Returns an int32 GPU tensor [nh] of chunks (no synchronisation)."""
    return (_ext or _native()).corey_select_chunk_device(r_dev, L, policy, seqlens, out)


def selective_scan_fwd_plan(B: int, D: int, N: int, chunk: int) -> int:
    return int(lib().selective_scan_fwd_plan(B, D, N, chunk))


def selective_scan_fwd_plan_steps(B: int, D: int, N: int, chunk: int) -> int:
    return int(lib().selective_scan_fwd_plan_steps(B, D, N, chunk))


def selective_scan_fwd_plan_split(B: int, D: int, N: int, chunk: int) -> int:
    return int(lib().selective_scan_fwd_plan_split(B, D, N, chunk))


def selective_scan_fwd_workspace(B: int, N: int, L: int) -> int:
    return int(lib().selective_scan_fwd_workspace(B, N, L))


COREY_SCAN_GENERAL_A = 1
COREY_SCAN_ONE_CHUNK = 2
COREY_SCAN_WHOLE_ROWS = 4


def selective_scan_fwd(u, delta, A, Bm, Cm, Dv=None, z=None, delta_bias=None, delta_softplus=True, h0=None,
                       seqlens=None, chunk: int = 512, chunks_dev=None, y=None, last_state=None, workspace=None,
                       general_a: bool = False, route: DeferredRoute | None = None, whole_rows: bool = False):
    """Tensors as in include/corey.h.  Returns (y, last_state); enqueues on torch's current stream.
    `workspace`: uint8 GPU tensor of selective_scan_fwd_workspace(B, N, L) bytes (allocated here if omitted).
    `general_a`: COREY_SCAN_GENERAL_A, i.e. never take the fast path for A[d, n] = (n + 1) A[d, 0].
    `chunks_dev` of one entry for a batch of several sequences is passed with COREY_SCAN_ONE_CHUNK.
    `whole_rows`: COREY_SCAN_WHOLE_ROWS, i.e. never share a channel's states between two rows of lanes.
    `route`: the ticket of corey_route_device_deferred; the call is then selective_scan_fwd_routed (no chunks_dev)."""
    return (_ext or _native()).selective_scan_fwd(u, delta, A, Bm, Cm, Dv, z, delta_bias, delta_softplus, h0, seqlens, chunk, chunks_dev, y,
                                                  last_state, workspace, general_a, route, whole_rows)
