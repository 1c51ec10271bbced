"""ctypes binding of the C ABI declared in include/grace_moe.h."""
from __future__ import annotations

import ctypes as C
import importlib
import os
import warnings
from typing import Optional, Sequence, Tuple

import numpy as np
import torch

from . import build as _build

GRACE_F32, GRACE_BF16 = 0, 1
GRACE_POLICY_TAR, GRACE_POLICY_WRR = 0, 1
SHARE_STATE_INTS = 8      # GRACE_SHARE_STATE_INTS
_STATUS = {0: "GRACE_OK", -1: "GRACE_EINVAL", -2: "GRACE_ESHAPE", -3: "GRACE_ETABLE", -4: "GRACE_ENOMEM",
           -5: "GRACE_EHIP"}

EXPORTS = ("grace_table_validate", "grace_table_create", "grace_table_destroy", "grace_table_info",
           "grace_table_instances", "grace_table_local_experts", "grace_table_set_fold_limits", "grace_workspace_bytes",
           "grace_route",
           "grace_permute", "grace_permute_rows", "grace_route_permute", "grace_route_permute_static", "grace_send_lists", "grace_send_lists_fresh", "grace_expert_ffn", "grace_expert_ffn_up",
           "grace_expert_ffn_down", "grace_expert_ffn_down_fresh", "grace_expert_ffn_up_share", "grace_expert_ffn_up_share_scatter", "grace_expert_ffn_down_share",
           "grace_shared_ffn", "grace_shared_ffn_up", "grace_shared_ffn_down", "grace_shared_ffn_up_scatter", "grace_combine", "grace_combine_share", "grace_mfma_sustained",
           "grace_ffn_kernel", "grace_ffn_carries_rows",
           "grace_dispatch_ffn_up_share", "grace_dispatch_ffn_down_share", "grace_dispatch_joins_ffn", "grace_expert_shared_ffn_up_scatter", "grace_expert_shared_ffn_down", "grace_ffn_joins_shared",
           "grace_last_error")

_lib: Optional[C.CDLL] = None
_calls = None   # the module of the calls that allocate their outputs (csrc/torch_calls.cpp), False: it cannot be had


class GraceError(RuntimeError):
    def __init__(self, status: int, text: str):
        super().__init__(f"{_STATUS.get(status, status)}: {text}")
        self.status = status


def library_path() -> str:
    return _build.LIB


def load_library() -> C.CDLL:
    """Load the in-tree shared library.  It is built first when it is absent or older than any of
    its sources, so a forgotten rebuild cannot put yesterday's kernels under today's tests; where the
    sources are newer and no compiler is available the call fails instead of loading the old code."""
    global _lib
    if _lib is not None:
        return _lib
    if _build.is_stale():
        _build.build_library()
    lib = C.CDLL(_build.LIB)
    vp, i32, u64 = C.c_void_p, C.c_int32, C.c_size_t
    lib.grace_last_error.restype = C.c_char_p
    lib.grace_last_error.argtypes = []
    lib.grace_table_validate.argtypes = [i32, i32, i32, vp, vp, vp, vp]
    lib.grace_table_create.argtypes = [C.POINTER(vp), i32, i32, i32, vp, vp, vp, vp, vp]
    lib.grace_table_destroy.argtypes = [vp]
    lib.grace_table_info.argtypes = [vp] + [C.POINTER(i32)] * 5
    lib.grace_table_instances.argtypes = [vp, vp, vp, vp]
    lib.grace_table_local_experts.argtypes = [vp, i32, vp, C.POINTER(i32)]
    lib.grace_table_set_fold_limits.argtypes = [vp, i32, i32]
    lib.grace_workspace_bytes.restype = u64
    lib.grace_workspace_bytes.argtypes = [i32] * 7 + [C.c_int]
    lib.grace_route.argtypes = [vp, i32, C.c_int, vp, i32, i32, i32, i32, vp, vp, vp, vp, vp, vp, vp, vp]
    lib.grace_permute.argtypes = [vp, vp, i32, i32, vp, i32, C.c_int, vp, vp, vp, vp, vp, vp, vp, vp]
    lib.grace_permute_rows.argtypes = [vp, vp, i32, i32, i32, C.c_int, vp, vp]
    lib.grace_route_permute.argtypes = [vp, i32, C.c_int, vp, i32, i32, i32, i32, vp, vp, vp, vp, vp, vp,
                                        vp, i32, C.c_int, vp, vp, vp, vp, vp, vp, vp, vp]
    lib.grace_route_permute_static.argtypes = [vp, i32, C.c_int, vp, i32, i32, i32, i32, vp, vp, vp, vp, vp, vp,
                                               vp, i32, C.c_int, vp, vp, vp, vp, vp, vp, vp]
    lib.grace_send_lists.argtypes = [vp, i32, vp, i32, i32, vp, vp, vp, vp, vp, vp, vp, vp]
    lib.grace_send_lists_fresh.argtypes = lib.grace_send_lists.argtypes
    lib.grace_expert_ffn.argtypes = [vp, i32, vp, vp, i32, i32, i32, i32, C.c_int, vp, vp, vp, vp, vp, vp]
    lib.grace_expert_ffn_up.argtypes = [vp, i32, vp, vp, i32, i32, i32, i32, C.c_int, vp, vp, vp, vp]
    lib.grace_expert_ffn_down.argtypes = [vp, i32, vp, i32, i32, i32, i32, C.c_int, vp, vp, vp, vp]
    lib.grace_expert_ffn_down_fresh.argtypes = lib.grace_expert_ffn_down.argtypes
    lib.grace_expert_ffn_up_share.argtypes = [vp, i32, vp, vp, i32, i32, i32, i32, C.c_int, vp, vp, vp, vp, vp]
    lib.grace_expert_ffn_up_share_scatter.argtypes = [vp, i32, vp, vp, vp, vp, vp, i32, i32, i32, i32, C.c_int, vp, vp, vp, vp, vp]
    lib.grace_expert_ffn_down_share.argtypes = [vp, i32, vp, i32, i32, i32, i32, C.c_int, vp, vp, vp, vp, vp]
    lib.grace_shared_ffn.argtypes = [vp, i32, i32, i32, i32, C.c_int, vp, vp, vp, vp, vp, vp]
    lib.grace_shared_ffn_up.argtypes = [vp, i32, i32, i32, i32, C.c_int, vp, vp, vp, vp]
    lib.grace_shared_ffn_up_scatter.argtypes = [vp, i32, i32, i32, i32, C.c_int, vp, vp, vp, vp, i32, vp, vp]
    lib.grace_shared_ffn_down.argtypes = [i32, i32, i32, i32, C.c_int, vp, vp, vp, vp]
    lib.grace_combine.argtypes = [vp, vp, vp, i32, i32, i32, C.c_int, vp, vp, vp]
    lib.grace_combine_share.argtypes = [vp, vp, vp, i32, i32, i32, C.c_int, vp, vp, vp, vp]
    lib.grace_mfma_sustained.argtypes = [i32, i32, C.POINTER(C.c_double), vp]
    lib.grace_ffn_kernel.argtypes = [i32] * 8 + [C.c_int, i32, C.POINTER(i32), C.POINTER(C.c_int64)]
    lib.grace_dispatch_ffn_up_share.argtypes = [vp, i32, C.c_int, vp, i32, i32, i32, i32, vp, vp, vp, vp, vp, vp, vp, i32, i32, i32, C.c_int,
                                                vp, vp, vp, vp, vp, vp, vp, vp, vp, vp, vp, vp, vp, vp]
    lib.grace_dispatch_ffn_down_share.argtypes = [vp, i32, vp, vp, vp, i32, i32, i32, i32, i32, C.c_int, vp, vp, vp, vp, vp, vp, vp, vp, vp]
    lib.grace_expert_shared_ffn_up_scatter.argtypes = [vp, i32, vp, vp, vp, vp, vp, i32, i32, i32, i32, i32, C.c_int, vp, vp, vp, vp, vp, vp, vp, vp]
    lib.grace_expert_shared_ffn_down.argtypes = [vp, i32, vp, i32, i32, i32, i32, i32, C.c_int, vp, vp, vp, vp, vp, vp, vp, vp]
    lib.grace_ffn_joins_shared.argtypes = [i32] * 8 + [C.c_int, i32, vp]
    lib.grace_dispatch_joins_ffn.argtypes = [vp, i32, i32, i32, i32, i32, i32, C.c_int, i32, vp]
    lib.grace_ffn_carries_rows.argtypes = [i32, i32, i32, i32, i32, i32, i32, C.c_int, i32, vp]
    for name in EXPORTS:
        if name not in ("grace_last_error", "grace_workspace_bytes"):
            getattr(lib, name).restype = C.c_int
    _lib = lib
    return lib


def grace_last_error() -> str:
    return load_library().grace_last_error().decode()


def _check(status: int) -> None:
    if status != 0:
        raise GraceError(status, grace_last_error())


def _made(result):
    """What a native call has made, or its error."""
    if isinstance(result, int):
        _check(result)
    return result


def _native():
    """The module of the calls that allocate their outputs, built first where it is absent or older than its source; None where it cannot be
    built (g++, Python's or torch's headers missing): these calls then go through Python, as those on the caller's buffers do."""
    global _calls
    if _calls is None:
        lib = load_library()
        try:
            if _build.calls_are_stale():
                _build.build_calls()
            calls = importlib.import_module("._torch_calls", __package__)
            calls.bind(*(C.cast(f, C.c_void_p).value for f in (lib.grace_workspace_bytes, lib.grace_route, lib.grace_permute, lib.grace_route_permute,
                                                               lib.grace_send_lists_fresh)))
        except (OSError, RuntimeError, ImportError) as e:
            warnings.warn(f"the binding's native calls are not available, calls that allocate go through Python: {e}")
            calls = False
        _calls = calls
    return _calls or None


def _host(a, dtype) -> np.ndarray:
    return np.ascontiguousarray(np.asarray(a), dtype=dtype)


def _hp(a: Optional[np.ndarray]):
    return None if a is None else a.ctypes.data_as(C.c_void_p)


# A call of three or four of these functions per batch of a deployment planner is bound by what happens here: addresses go
# to ctypes as integers, the stream's address is asked for without building a Stream object (route, send lists and
# dispatch order of 16384 tokens 82.6 -> 74.1 us), and calls that allocate all of their outputs are native (_torch_calls, 59.4 -> 41.8 us).
def _dp(t: Optional[torch.Tensor]):
    if t is None:
        return None
    if not t.is_cuda or not t.is_contiguous():
        raise ValueError("device tensors must be contiguous and live on the GPU")
    return t.data_ptr()


def _stream() -> int:
    # (_cuda_getDevice initialises the device on first use, as current_stream() does)
    return torch._C._cuda_getCurrentRawStream(torch._C._cuda_getDevice())


def _dtype_code(t: torch.Tensor) -> int:
    if t.dtype == torch.float32:
        return GRACE_F32
    if t.dtype == torch.bfloat16:
        return GRACE_BF16
    raise ValueError(f"unsupported dtype {t.dtype}")


def grace_table_validate(E, R, N, rank_node, poll_weight, inst_ptr, inst_rank) -> None:
    """Host-only validation of a placement table; raises GraceError."""
    a = (_host(rank_node, np.int32), _host(poll_weight, np.uint32), _host(inst_ptr, np.int32),
         _host(inst_rank, np.int32))
    _check(load_library().grace_table_validate(E, R, N, *[_hp(x) for x in a]))


def grace_workspace_bytes(T, E, k, I, d=0, f=0, n_shared=0, dt=GRACE_BF16) -> int:
    return int(load_library().grace_workspace_bytes(T, E, k, I, d, f, n_shared, dt))


class GraceTable:
    """Owns a grace_table (device copy on the current GPU)."""

    def __init__(self, E, R, N, rank_node, poll_weight, inst_ptr, inst_rank):
        lib = load_library()
        a = (_host(rank_node, np.int32), _host(poll_weight, np.uint32), _host(inst_ptr, np.int32),
             _host(inst_rank, np.int32))
        h = C.c_void_p()
        _check(lib.grace_table_create(C.byref(h), E, R, N, *[_hp(x) for x in a], _stream()))
        self._h = h
        v = [C.c_int32() for _ in range(5)]
        _check(lib.grace_table_info(h, *[C.byref(x) for x in v]))
        self.E, self.R, self.N, self.I, self.max_local_slots = (int(x.value) for x in v)

    @classmethod
    def from_placement(cls, pl) -> "GraceTable":
        return cls(pl.E, pl.R, pl.N, pl.rank_node, pl.poll_weight, pl.inst_ptr, pl.inst_rank)

    @property
    def handle(self):
        if self._h is None:
            raise ValueError("table was destroyed")
        return self._h

    def instances(self) -> Tuple[np.ndarray, np.ndarray, np.ndarray]:
        """(inst_expert [I], inst_rank [I], rank_ptr [R+1]) in dispatch order."""
        ie, ir, rp = np.empty(self.I, np.int32), np.empty(self.I, np.int32), np.empty(self.R + 1, np.int32)
        _check(load_library().grace_table_instances(self.handle, _hp(ie), _hp(ir), _hp(rp)))
        return ie, ir, rp

    def local_experts(self, rank: int) -> np.ndarray:
        buf = np.empty(max(self.max_local_slots, 1), np.int32)
        n = C.c_int32()
        _check(load_library().grace_table_local_experts(self.handle, rank, _hp(buf), C.byref(n)))
        return buf[:n.value].copy()

    def set_fold_limits(self, one_level_max: int = -1, two_level_max: int = -1) -> None:
        """Switch points of the index kernels' prefix-count algorithms for calls with this table
        (negative: defaults); see grace_moe.h."""
        _check(load_library().grace_table_set_fold_limits(self.handle, one_level_max, two_level_max))

    def destroy(self) -> None:
        if getattr(self, "_h", None) is not None:
            h, self._h = self._h, None
            _check(load_library().grace_table_destroy(h))

    def __del__(self):
        try:
            self.destroy()
        except Exception:
            pass


def _ws(ws: Optional[torch.Tensor], nbytes: int, device) -> torch.Tensor:
    if ws is None:
        ws = torch.empty(max(nbytes, 256), dtype=torch.uint8, device=device)
    elif ws.numel() * ws.element_size() < nbytes:
        raise ValueError(f"workspace too small: need {nbytes} bytes")
    return ws


def _need_ws(ws: Optional[torch.Tensor], nbytes: int) -> None:
    """A workspace that a later call reads as well: the caller's."""
    if ws is None:
        raise ValueError(f"workspace missing: need {nbytes} bytes")
    _ws(ws, nbytes, ws.device)


def _need(t: Optional[torch.Tensor], name: str, dtype: torch.dtype, numel: int) -> None:
    """A caller's tensor that a kernel reads or writes `numel` entries of."""
    if t is None or t.dtype != dtype or t.numel() < numel:
        raise ValueError(f"{name} must hold {numel} {str(dtype).replace('torch.', '')}")


def grace_route(table: GraceTable, local_rank: int, logits: torch.Tensor, k: int, renorm: int = 1,
                rr_in: Optional[torch.Tensor] = None, rr_out: Optional[torch.Tensor] = None,
                ws: Optional[torch.Tensor] = None, out=None, policy: int = GRACE_POLICY_TAR):
    """-> (topk_expert [T,k] i32, topk_weight [T,k] f32, topk_inst [T,k] i32, expert_count [E] i32)."""
    native = _native() if out is None and ws is None else None
    if native:
        return _made(native.route(table.handle.value, table.I, local_rank, logits, k, renorm, rr_in, rr_out, policy, _stream()))
    T, E = logits.shape
    dev = logits.device
    if logits.dtype != torch.float32:
        raise ValueError("logits must be float32")
    if out is None:
        out = (torch.empty((T, k), dtype=torch.int32, device=dev), torch.empty((T, k), dtype=torch.float32, device=dev),
               torch.empty((T, k), dtype=torch.int32, device=dev), torch.empty((E,), dtype=torch.int32, device=dev))
    te, tw, ti, cnt = out
    ws = _ws(ws, grace_workspace_bytes(T, E, max(k, 1), table.I), dev)
    _check(load_library().grace_route(table.handle, local_rank, policy, _dp(logits), T, E, k, renorm, _dp(rr_in), _dp(rr_out),
                                      _dp(te), _dp(tw), _dp(ti), _dp(cnt), _dp(ws), _stream()))
    return te, tw, ti, cnt


def grace_permute(table: GraceTable, topk_inst: torch.Tensor, x: Optional[torch.Tensor], ws: Optional[torch.Tensor] = None,
                  out=None, xp: Optional[torch.Tensor] = None):
    """-> (perm_pos, perm_src, inst_off, rank_off, node_off, xp)."""
    native = _native() if out is None and ws is None and xp is None else None
    if native:
        return _made(native.permute(table.handle.value, table.E, table.I, table.R, table.N, topk_inst, x, _stream()))
    T, k = topk_inst.shape
    dev = topk_inst.device
    if out is None:
        i32 = dict(dtype=torch.int32, device=dev)
        out = (torch.empty(T * k, **i32), torch.empty(T * k, **i32), torch.empty(table.I + 1, **i32),
               torch.empty(table.R + 1, **i32), torch.empty(table.N + 1, **i32))
    pos, src, ioff, roff, noff = out
    d, dt = 0, GRACE_BF16
    if x is not None:
        d, dt = x.shape[1], _dtype_code(x)
        if xp is None:
            xp = torch.empty((T * k, d), dtype=x.dtype, device=dev)
    ws = _ws(ws, grace_workspace_bytes(T, table.E, k, table.I), dev)
    _check(load_library().grace_permute(table.handle, _dp(topk_inst), T, k, _dp(x), d, dt, _dp(pos), _dp(src), _dp(ioff),
                                        _dp(roff), _dp(noff), _dp(xp) if x is not None else None, _dp(ws), _stream()))
    return pos, src, ioff, roff, noff, xp


def grace_route_permute(table: GraceTable, local_rank: int, logits: torch.Tensor, k: int, x: Optional[torch.Tensor],
                        renorm: int = 1, rr_in: Optional[torch.Tensor] = None, rr_out: Optional[torch.Tensor] = None,
                        ws: Optional[torch.Tensor] = None, policy: int = GRACE_POLICY_TAR):
    """grace_route and grace_permute as one call with fewer launches (see grace_moe.h).
    -> ((topk_expert, topk_weight, topk_inst, expert_count), (perm_pos, perm_src, inst_off, rank_off, node_off, xp))."""
    native = _native() if ws is None else None
    if native:
        return _made(native.route_permute(table.handle.value, table.I, table.R, table.N, local_rank, logits, k, x, renorm, rr_in, rr_out,
                                          policy, _stream()))
    T, E = logits.shape
    dev = logits.device
    if logits.dtype != torch.float32:
        raise ValueError("logits must be float32")
    i32 = dict(dtype=torch.int32, device=dev)
    te, tw = torch.empty((T, k), **i32), torch.empty((T, k), dtype=torch.float32, device=dev)
    ti, cnt = torch.empty((T, k), **i32), torch.empty((E,), **i32)
    pos, src = torch.empty(T * k, **i32), torch.empty(T * k, **i32)
    ioff, roff, noff = torch.empty(table.I + 1, **i32), torch.empty(table.R + 1, **i32), torch.empty(table.N + 1, **i32)
    d, dt, xp = 0, GRACE_BF16, None
    if x is not None:
        d, dt = x.shape[1], _dtype_code(x)
        xp = torch.empty((T * k, d), dtype=x.dtype, device=dev)
    ws = _ws(ws, grace_workspace_bytes(T, E, max(k, 1), table.I), dev)
    _check(load_library().grace_route_permute(table.handle, local_rank, policy, _dp(logits), T, E, k, renorm, _dp(rr_in),
                                              _dp(rr_out), _dp(te), _dp(tw), _dp(ti), _dp(cnt), _dp(x), d, dt, _dp(pos),
                                              _dp(src), _dp(ioff), _dp(roff), _dp(noff),
                                              _dp(xp) if x is not None else None, _dp(ws), _stream()))
    return (te, tw, ti, cnt), (pos, src, ioff, roff, noff, xp)


def grace_route_permute_static(table: GraceTable, local_rank: int, logits: torch.Tensor, k: int, x: Optional[torch.Tensor],
                               renorm: int = 1, rr_in: Optional[torch.Tensor] = None, rr_out: Optional[torch.Tensor] = None,
                               policy: int = GRACE_POLICY_TAR, out=None):
    """grace_route_permute on the library's static scratch instead of a workspace (see grace_moe.h).
    `out` = ((topk_expert, topk_weight, topk_inst, expert_count), (perm_pos, perm_src, inst_off, rank_off,
    node_off, xp)) reuses the caller's output tensors; the C call itself allocates nothing."""
    T, E = logits.shape
    dev = logits.device
    if logits.dtype != torch.float32:
        raise ValueError("logits must be float32")
    d, dt = (0, GRACE_BF16) if x is None else (x.shape[1], _dtype_code(x))
    if out is None:
        i32 = dict(dtype=torch.int32, device=dev)
        out = ((torch.empty((T, k), **i32), torch.empty((T, k), dtype=torch.float32, device=dev), torch.empty((T, k), **i32),
                torch.empty((E,), **i32)),
               (torch.empty(T * k, **i32), torch.empty(T * k, **i32), torch.empty(table.I + 1, **i32),
                torch.empty(table.R + 1, **i32), torch.empty(table.N + 1, **i32),
                None if x is None else torch.empty((T * k, d), dtype=x.dtype, device=dev)))
    (te, tw, ti, cnt), (pos, src, ioff, roff, noff, xp) = out
    _check(load_library().grace_route_permute_static(table.handle, local_rank, policy, _dp(logits), T, E, k, renorm, _dp(rr_in),
                                                     _dp(rr_out), _dp(te), _dp(tw), _dp(ti), _dp(cnt), _dp(x), d, dt, _dp(pos),
                                                     _dp(src), _dp(ioff), _dp(roff), _dp(noff),
                                                     _dp(xp) if x is not None else None, _stream()))
    return out


def grace_send_lists(table: GraceTable, local_rank: int, topk_inst: torch.Tensor, ws: Optional[torch.Tensor] = None):
    """-> (rank_send_ptr [R+1], rank_send_tok [T*k], node_send_ptr [N+1], node_send_tok [T*k], expand [T*k],
    traffic [4] int64); see grace_moe.h."""
    native = _native() if ws is None else None
    if native:
        return _made(native.send_lists(table.handle.value, table.E, table.I, table.R, table.N, local_rank, topk_inst, _stream()))
    T, k = topk_inst.shape
    dev = topk_inst.device
    i32 = dict(dtype=torch.int32, device=dev)
    rp, rt = torch.empty(table.R + 1, **i32), torch.empty(T * k, **i32)
    np_, nt = torch.empty(table.N + 1, **i32), torch.empty(T * k, **i32)
    ex = torch.empty(T * k, **i32)
    tr = torch.empty(4, dtype=torch.int64, device=dev)
    _send_lists_fresh(table, local_rank, topk_inst, rp, rt, np_, nt, ex, tr, ws)
    return rp, rt, np_, nt, ex, tr


def grace_send_lists_fresh(table: GraceTable, local_rank: int, topk_inst: torch.Tensor, out, ws: Optional[torch.Tensor] = None) -> None:
    """grace_send_lists into the caller's tensors, all of whose entries are written (-1 past the ends of the lists);
    `out` as grace_send_lists returns it, traffic may be None."""
    T, k = topk_inst.shape
    rp, rt, np_, nt, ex, tr = out
    for t, name, n in ((rp, "rank_send_ptr", table.R + 1), (rt, "rank_send_tok", T * k), (np_, "node_send_ptr", table.N + 1),
                       (nt, "node_send_tok", T * k), (ex, "expand", T * k)):
        _need(t, name, torch.int32, n)
    if tr is not None:
        _need(tr, "traffic", torch.int64, 4)
    _send_lists_fresh(table, local_rank, topk_inst, rp, rt, np_, nt, ex, tr, ws)


def _send_lists_fresh(table, local_rank, topk_inst, rp, rt, np_, nt, ex, tr, ws) -> None:
    T, k = topk_inst.shape
    ws = _ws(ws, grace_workspace_bytes(T, table.E, k, table.I), topk_inst.device)
    _check(load_library().grace_send_lists_fresh(table.handle, local_rank, _dp(topk_inst), T, k, _dp(rp), _dp(rt), _dp(np_),
                                                 _dp(nt), _dp(ex), _dp(tr), _dp(ws), _stream()))


def grace_expert_ffn(table: GraceTable, rank: int, xp: torch.Tensor, inst_off: torch.Tensor, T: int, k: int,
                     w_gate: torch.Tensor, w_up: torch.Tensor, w_down: torch.Tensor, y: Optional[torch.Tensor] = None,
                     ws: Optional[torch.Tensor] = None) -> torch.Tensor:
    """y [T*k, d]; only the rows of `rank` are written (a fresh y starts as zeros)."""
    d = xp.shape[1]
    dt = _dtype_code(xp)
    S = w_gate.shape[0]
    f = w_gate.shape[1] if S > 0 else (w_down.shape[2] if w_down.dim() == 3 else 8)
    if S > 0 and (tuple(w_gate.shape) != (S, f, d) or tuple(w_up.shape) != (S, f, d) or tuple(w_down.shape) != (S, d, f)):
        raise ValueError("weights must be w_gate/w_up [S,f,d] and w_down [S,d,f]")
    for w in (w_gate, w_up, w_down):
        if w.dtype != xp.dtype:
            raise ValueError("weights and activations must share one dtype")
    ws = _ws(ws, grace_workspace_bytes(T, table.E, k, table.I, d, f, 0, dt), xp.device)
    if y is None and S > 0 and d * xp.element_size() % 16 == 0:
        # the down projection's launch zeroes the rows of other ranks (8000 rows of 4 KB, none of them another rank's:
        # 9 us for a fill of all of them)
        y = torch.empty((T * k, d), dtype=xp.dtype, device=xp.device)
        lib = load_library()
        _check(lib.grace_expert_ffn_up(table.handle, rank, _dp(xp), _dp(inst_off), T, k, d, f, dt, _dp(w_gate), _dp(w_up), _dp(ws),
                                       _stream()))
        _check(lib.grace_expert_ffn_down_fresh(table.handle, rank, _dp(inst_off), T, k, d, f, dt, _dp(w_down), _dp(y), _dp(ws),
                                               _stream()))
        return y
    if y is None:
        y = torch.zeros((T * k, d), dtype=xp.dtype, device=xp.device)
    _check(load_library().grace_expert_ffn(table.handle, rank, _dp(xp), _dp(inst_off), T, k, d, f, dt,
                                           _dp(w_gate) if S else None, _dp(w_up) if S else None,
                                           _dp(w_down) if S else None, _dp(y), _dp(ws), _stream()))
    return y


def grace_expert_ffn_up(table: GraceTable, rank: int, xp: torch.Tensor, inst_off: torch.Tensor, T: int, k: int,
                        w_gate: torch.Tensor, w_up: torch.Tensor, ws: torch.Tensor) -> None:
    S, f, d = w_gate.shape
    _check(load_library().grace_expert_ffn_up(table.handle, rank, _dp(xp), _dp(inst_off), T, k, d, f, _dtype_code(xp),
                                              _dp(w_gate) if S else None, _dp(w_up) if S else None, _dp(ws), _stream()))


def grace_expert_ffn_down(table: GraceTable, rank: int, inst_off: torch.Tensor, T: int, k: int, w_down: torch.Tensor,
                          y: torch.Tensor, ws: torch.Tensor) -> None:
    S, d, f = w_down.shape
    _check(load_library().grace_expert_ffn_down(table.handle, rank, _dp(inst_off), T, k, d, f, _dtype_code(y),
                                                _dp(w_down) if S else None, _dp(y), _dp(ws), _stream()))


def grace_expert_ffn_down_fresh(table: GraceTable, rank: int, inst_off: torch.Tensor, T: int, k: int, w_down: torch.Tensor,
                                y: torch.Tensor, ws: torch.Tensor) -> None:
    """grace_expert_ffn_down that also zeroes the rows of other ranks; see grace_moe.h."""
    S, d, f = w_down.shape
    _check(load_library().grace_expert_ffn_down_fresh(table.handle, rank, _dp(inst_off), T, k, d, f, _dtype_code(y),
                                                      _dp(w_down) if S else None, _dp(y), _dp(ws), _stream()))


def grace_expert_ffn_up_share(table: GraceTable, rank: int, xp: torch.Tensor, inst_off: torch.Tensor, T: int, k: int,
                              w_gate: torch.Tensor, w_up: torch.Tensor, state: torch.Tensor, ws: torch.Tensor) -> None:
    """grace_expert_ffn_up that also records the rank's row range of this step in `state` (first half of
    the pair with grace_expert_ffn_down_share); see grace_moe.h."""
    if state.dtype != torch.int32 or state.numel() < SHARE_STATE_INTS:
        raise ValueError(f"state must hold {SHARE_STATE_INTS} int32")
    S, f, d = w_gate.shape
    _check(load_library().grace_expert_ffn_up_share(table.handle, rank, _dp(xp), _dp(inst_off), T, k, d, f, _dtype_code(xp),
                                                    _dp(w_gate) if S else None, _dp(w_up) if S else None, _dp(state),
                                                    _dp(ws), _stream()))


def grace_expert_ffn_up_share_scatter(table: GraceTable, rank: int, x: torch.Tensor, perm_pos: torch.Tensor, perm_src: torch.Tensor,
                                      xp: torch.Tensor, inst_off: torch.Tensor, k: int, w_gate: torch.Tensor, w_up: torch.Tensor,
                                      state: torch.Tensor, ws: torch.Tensor) -> None:
    """grace_permute_rows (rows of x into xp) and grace_expert_ffn_up_share on them as one call; see grace_moe.h."""
    if state.dtype != torch.int32 or state.numel() < SHARE_STATE_INTS:
        raise ValueError(f"state must hold {SHARE_STATE_INTS} int32")
    S, f, d = w_gate.shape
    T = x.shape[0]
    if tuple(x.shape) != (T, d) or tuple(w_up.shape) != (S, f, d) or w_gate.dtype != x.dtype or w_up.dtype != x.dtype:
        raise ValueError("x must be [T,d], w_gate and w_up [S,f,d], of one dtype")
    for t, name, n in ((perm_pos, "perm_pos", T * k), (perm_src, "perm_src", T * k), (inst_off, "inst_off", table.I + 1)):
        _need(t, name, torch.int32, n)
    _need(xp, "xp", x.dtype, T * k * d)
    ws = _ws(ws, grace_workspace_bytes(T, table.E, k, table.I, d, f, 0, _dtype_code(x)), x.device)
    _check(load_library().grace_expert_ffn_up_share_scatter(table.handle, rank, _dp(x), _dp(perm_pos), _dp(perm_src), _dp(xp), _dp(inst_off),
                                                            T, k, d, f, _dtype_code(x), _dp(w_gate) if S else None,
                                                            _dp(w_up) if S else None, _dp(state), _dp(ws), _stream()))


def grace_expert_ffn_down_share(table: GraceTable, rank: int, inst_off: torch.Tensor, T: int, k: int, w_down: torch.Tensor,
                                y: torch.Tensor, state: torch.Tensor, ws: torch.Tensor) -> None:
    """grace_expert_ffn_down that also zeroes the rows the previous step (same `state`: SHARE_STATE_INTS
    int32 on the device, zero before the first step, kept by grace_expert_ffn_up_share) wrote outside the
    rank's current row range; see grace_moe.h."""
    if state.dtype != torch.int32 or state.numel() < SHARE_STATE_INTS:
        raise ValueError(f"state must hold {SHARE_STATE_INTS} int32")
    S, d, f = w_down.shape
    _check(load_library().grace_expert_ffn_down_share(table.handle, rank, _dp(inst_off), T, k, d, f, _dtype_code(y),
                                                      _dp(w_down) if S else None, _dp(y), _dp(state), _dp(ws), _stream()))


def _shared_weights(shared, n: int, d: int, f: int, dtype: torch.dtype) -> int:
    """Checked shared weights (`n` of them: gate and up [n,f,d], or down [n,d,f]); how many experts they are."""
    if shared is None:
        return 0
    want = (shared[0].shape[0],) + ((f, d) if n == 2 else (d, f))
    if any(tuple(w.shape) != want or w.dtype != dtype for w in shared):
        raise ValueError("shared weights must be [n,f,d] (gate, up) and [n,d,f] (down) of one dtype")
    return want[0]


def grace_dispatch_ffn_up_share(table: GraceTable, local_rank: int, logits: torch.Tensor, k: int, x: torch.Tensor, w_gate: torch.Tensor,
                                w_up: torch.Tensor, state: torch.Tensor, ws: torch.Tensor, renorm: int = 1,
                                rr_in: Optional[torch.Tensor] = None, rr_out: Optional[torch.Tensor] = None,
                                policy: int = GRACE_POLICY_TAR, shared: Optional[Tuple[torch.Tensor, torch.Tensor]] = None,
                                ws_shared: Optional[torch.Tensor] = None):
    """Dispatch and gate+up projections of the local rank as one call (one launch for the smallest batches), `shared` = the shared
    experts' (gate, up); the rest of the step is grace_dispatch_ffn_down_share.  -> what grace_route_permute returns; see grace_moe.h."""
    _need(state, "state", torch.int32, SHARE_STATE_INTS)
    T, E = logits.shape
    S, f, d = w_gate.shape
    if logits.dtype != torch.float32:
        raise ValueError("logits must be float32")
    if tuple(x.shape) != (T, d) or tuple(w_up.shape) != (S, f, d) or w_gate.dtype != x.dtype or w_up.dtype != x.dtype:
        raise ValueError("x must be [T,d], w_gate and w_up [S,f,d], of one dtype")
    dt, dev = _dtype_code(x), logits.device
    n_shared = _shared_weights(shared, 2, d, f, x.dtype)
    _need_ws(ws, grace_workspace_bytes(T, E, max(k, 1), table.I, d, f, 0, dt))
    if n_shared:
        _need_ws(ws_shared, grace_workspace_bytes(T, 1, 1, 1, d, f, n_shared, dt))
    i32 = dict(dtype=torch.int32, device=dev)
    te, tw = torch.empty((T, k), **i32), torch.empty((T, k), dtype=torch.float32, device=dev)
    ti, cnt = torch.empty((T, k), **i32), torch.empty((E,), **i32)
    pos, src = torch.empty(T * k, **i32), torch.empty(T * k, **i32)
    ioff, roff, noff = torch.empty(table.I + 1, **i32), torch.empty(table.R + 1, **i32), torch.empty(table.N + 1, **i32)
    xp = torch.empty((T * k, d), dtype=x.dtype, device=dev)
    sg, su = shared if n_shared else (None, None)
    _check(load_library().grace_dispatch_ffn_up_share(
        table.handle, local_rank, policy, _dp(logits), T, E, k, renorm, _dp(rr_in), _dp(rr_out), _dp(te), _dp(tw), _dp(ti), _dp(cnt), _dp(x), d,
        f, n_shared, dt, _dp(pos), _dp(src), _dp(ioff), _dp(roff), _dp(noff), _dp(xp), _dp(w_gate) if S else None, _dp(w_up) if S else None,
        _dp(sg), _dp(su), _dp(state), _dp(ws), _dp(ws_shared), _stream()))
    return (te, tw, ti, cnt), (pos, src, ioff, roff, noff, xp)


def grace_dispatch_ffn_down_share(table: GraceTable, rank: int, inst_off: torch.Tensor, perm_pos: torch.Tensor, topk_weight: torch.Tensor,
                                  w_down: torch.Tensor, y: torch.Tensor, state: torch.Tensor, ws: torch.Tensor,
                                  shared_down: Optional[torch.Tensor] = None, y_shared: Optional[torch.Tensor] = None,
                                  ws_shared: Optional[torch.Tensor] = None, out: Optional[torch.Tensor] = None) -> torch.Tensor:
    """Down projections and combine behind grace_dispatch_ffn_up_share -> out [T,d]; see grace_moe.h."""
    _need(state, "state", torch.int32, SHARE_STATE_INTS)
    T, k = topk_weight.shape
    S, d, f = w_down.shape
    _need(topk_weight, "topk_weight", torch.float32, T * k)
    _need(perm_pos, "perm_pos", torch.int32, T * k)
    _need(inst_off, "inst_off", torch.int32, table.I + 1)
    _need(y, "y", w_down.dtype, T * k * d)
    n_shared, dt = _shared_weights(None if shared_down is None else (shared_down,), 1, d, f, w_down.dtype), _dtype_code(w_down)
    _need_ws(ws, grace_workspace_bytes(T, table.E, k, table.I, d, f, 0, dt))
    if n_shared:
        _need(y_shared, "y_shared", w_down.dtype, T * d)
        _need_ws(ws_shared, grace_workspace_bytes(T, 1, 1, 1, d, f, n_shared, dt))
    if out is None:
        out = torch.empty((T, d), dtype=y.dtype, device=y.device)
    _need(out, "out", w_down.dtype, T * d)
    _check(load_library().grace_dispatch_ffn_down_share(
        table.handle, rank, _dp(inst_off), _dp(perm_pos), _dp(topk_weight), T, k, d, f, n_shared, dt, _dp(w_down) if S else None,
        _dp(shared_down), _dp(y), _dp(y_shared), _dp(state), _dp(ws), _dp(ws_shared), _dp(out), _stream()))
    return out


def grace_dispatch_joins_ffn(table: GraceTable, local_rank: int, T: int, k: int, d: int, f: int, dt: int = GRACE_BF16, n_cu: int = 0,
                             n_shared: int = 0) -> int:
    """Does one launch do the dispatch and the experts' gate+up projection: 0, no; 1, yes; 2, and one the down projections and combine."""
    joined = C.c_int32()
    _check(load_library().grace_dispatch_joins_ffn(table.handle, local_rank, T, k, d, f, n_shared, dt, n_cu, C.byref(joined)))
    return joined.value


def grace_shared_ffn(x: torch.Tensor, w_gate: torch.Tensor, w_up: torch.Tensor, w_down: torch.Tensor,
                     y_shared: Optional[torch.Tensor] = None, ws: Optional[torch.Tensor] = None) -> torch.Tensor:
    T, d = x.shape
    n_shared, f, _ = w_gate.shape
    dt = _dtype_code(x)
    if tuple(w_up.shape) != (n_shared, f, d) or tuple(w_down.shape) != (n_shared, d, f):
        raise ValueError("weights must be w_gate/w_up [n,f,d] and w_down [n,d,f]")
    if y_shared is None:
        y_shared = torch.empty((T, d), dtype=x.dtype, device=x.device)
    ws = _ws(ws, grace_workspace_bytes(T, 1, 1, 1, d, f, n_shared, dt), x.device)
    _check(load_library().grace_shared_ffn(_dp(x), T, d, f, n_shared, dt, _dp(w_gate), _dp(w_up), _dp(w_down),
                                           _dp(y_shared), _dp(ws), _stream()))
    return y_shared


def grace_shared_ffn_up(x: torch.Tensor, w_gate: torch.Tensor, w_up: torch.Tensor, ws: torch.Tensor) -> None:
    """First launch of grace_shared_ffn: the hidden activation of all T rows into ws; see grace_moe.h."""
    T, d = x.shape
    n_shared, f, _ = w_gate.shape
    if tuple(w_up.shape) != (n_shared, f, d):
        raise ValueError("weights must be w_gate/w_up [n,f,d]")
    _check(load_library().grace_shared_ffn_up(_dp(x), T, d, f, n_shared, _dtype_code(x), _dp(w_gate), _dp(w_up), _dp(ws),
                                              _stream()))


def grace_shared_ffn_down(w_down: torch.Tensor, ws: torch.Tensor, T: int,
                          y_shared: Optional[torch.Tensor] = None) -> torch.Tensor:
    """Second launch of grace_shared_ffn: reads the hidden activation grace_shared_ffn_up left in ws; see grace_moe.h."""
    n_shared, d, f = w_down.shape
    if y_shared is None:
        y_shared = torch.empty((T, d), dtype=w_down.dtype, device=w_down.device)
    _check(load_library().grace_shared_ffn_down(T, d, f, n_shared, _dtype_code(w_down), _dp(w_down), _dp(y_shared), _dp(ws),
                                                _stream()))
    return y_shared


def grace_permute_rows(x: torch.Tensor, perm_pos: torch.Tensor, k: int, xp: Optional[torch.Tensor] = None) -> torch.Tensor:
    """The row movement of grace_permute alone: xp[perm_pos[t*k+j]] = x[t]; see grace_moe.h."""
    T, d = x.shape
    if xp is None:
        xp = torch.empty((T * k, d), dtype=x.dtype, device=x.device)
    _check(load_library().grace_permute_rows(_dp(x), _dp(perm_pos), T, k, d, _dtype_code(x), _dp(xp), _stream()))
    return xp


def grace_shared_ffn_up_scatter(x: torch.Tensor, w_gate: torch.Tensor, w_up: torch.Tensor, ws: torch.Tensor,
                                perm_pos: torch.Tensor, k: int, xp: torch.Tensor) -> None:
    """grace_shared_ffn_up (hidden activation into ws) and grace_permute_rows (rows into xp) as one call; see
    grace_moe.h."""
    T, d = x.shape
    n_shared, f, _ = w_gate.shape
    _check(load_library().grace_shared_ffn_up_scatter(_dp(x), T, d, f, n_shared, _dtype_code(x), _dp(w_gate), _dp(w_up),
                                                      _dp(ws), _dp(perm_pos), k, _dp(xp), _stream()))


def grace_expert_shared_ffn_up_scatter(table: GraceTable, rank: int, x: torch.Tensor, perm_pos: torch.Tensor, perm_src: torch.Tensor,
                                       xp: torch.Tensor, inst_off: torch.Tensor, k: int, w_gate: torch.Tensor, w_up: torch.Tensor,
                                       shared_gate: torch.Tensor, shared_up: torch.Tensor, state: torch.Tensor, ws: torch.Tensor,
                                       ws_shared: torch.Tensor) -> None:
    """grace_shared_ffn_up_scatter and grace_expert_ffn_up_share as one call; see grace_moe.h."""
    _need(state, "state", torch.int32, SHARE_STATE_INTS)
    S, f, d = w_gate.shape
    T, n_shared, dt = x.shape[0], shared_gate.shape[0], _dtype_code(x)
    if tuple(x.shape) != (T, d) or tuple(w_up.shape) != (S, f, d) or tuple(shared_gate.shape) != (n_shared, f, d) or \
            tuple(shared_up.shape) != (n_shared, f, d) or any(w.dtype != x.dtype for w in (w_gate, w_up, shared_gate, shared_up)):
        raise ValueError("x must be [T,d], w_gate and w_up [S,f,d], shared ones [n,f,d], of one dtype")
    for t, name, n in ((perm_pos, "perm_pos", T * k), (perm_src, "perm_src", T * k), (inst_off, "inst_off", table.I + 1)):
        _need(t, name, torch.int32, n)
    _need(xp, "xp", x.dtype, T * k * d)
    _need_ws(ws, grace_workspace_bytes(T, table.E, k, table.I, d, f, 0, dt))
    _need_ws(ws_shared, grace_workspace_bytes(T, 1, 1, 1, d, f, n_shared, dt))
    _check(load_library().grace_expert_shared_ffn_up_scatter(
        table.handle, rank, _dp(x), _dp(perm_pos), _dp(perm_src), _dp(xp), _dp(inst_off), T, k, d, f, n_shared, dt, _dp(w_gate) if S else None,
        _dp(w_up) if S else None, _dp(shared_gate), _dp(shared_up), _dp(state), _dp(ws), _dp(ws_shared), _stream()))


def grace_expert_shared_ffn_down(table: GraceTable, rank: int, inst_off: torch.Tensor, T: int, k: int, w_down: torch.Tensor,
                                 shared_down: torch.Tensor, y: torch.Tensor, y_shared: torch.Tensor, state: torch.Tensor, ws: torch.Tensor,
                                 ws_shared: torch.Tensor) -> None:
    """grace_expert_ffn_down_share and grace_shared_ffn_down as one call; see grace_moe.h."""
    _need(state, "state", torch.int32, SHARE_STATE_INTS)
    S, d, f = w_down.shape
    _need(y, "y", w_down.dtype, T * k * d)
    _need(y_shared, "y_shared", w_down.dtype, T * d)
    if tuple(shared_down.shape[1:]) != (d, f) or shared_down.dtype != w_down.dtype:
        raise ValueError("shared_down must be [n,d,f] of the dtype of w_down")
    n_shared, dt = shared_down.shape[0], _dtype_code(w_down)
    _need(inst_off, "inst_off", torch.int32, table.I + 1)
    _need_ws(ws, grace_workspace_bytes(T, table.E, k, table.I, d, f, 0, dt))
    _need_ws(ws_shared, grace_workspace_bytes(T, 1, 1, 1, d, f, n_shared, dt))
    _check(load_library().grace_expert_shared_ffn_down(
        table.handle, rank, _dp(inst_off), T, k, d, f, n_shared, dt, _dp(w_down) if S else None, _dp(shared_down),
        _dp(y), _dp(y_shared), _dp(state), _dp(ws), _dp(ws_shared), _stream()))


def grace_ffn_joins_shared(up: bool, T: int, d: int, f: int, n_shared: int, dt: int = GRACE_BF16, *, k: int = 1, S: int = 1, I: int = 1,
                           n_cu: int = 0) -> bool:
    """Does one launch do the experts' and the shared experts' projection (see grace_moe.h)?"""
    joined = C.c_int32()
    _check(load_library().grace_ffn_joins_shared(int(up), T, k, d, f, n_shared, S, I, dt, n_cu, C.byref(joined)))
    return bool(joined.value)


def grace_combine(y: torch.Tensor, perm_pos: torch.Tensor, topk_weight: torch.Tensor,
                  y_shared: Optional[torch.Tensor] = None, out: Optional[torch.Tensor] = None) -> torch.Tensor:
    T, k = topk_weight.shape
    d = y.shape[1]
    if out is None:
        out = torch.empty((T, d), dtype=y.dtype, device=y.device)
    _check(load_library().grace_combine(_dp(y), _dp(perm_pos), _dp(topk_weight), T, k, d, _dtype_code(y), _dp(y_shared),
                                        _dp(out), _stream()))
    return out


def grace_combine_share(y: torch.Tensor, perm_pos: torch.Tensor, topk_weight: torch.Tensor, state: torch.Tensor,
                        y_shared: Optional[torch.Tensor] = None, out: Optional[torch.Tensor] = None) -> torch.Tensor:
    """grace_combine of the rank share that grace_expert_ffn_up_share / _down_share with `state` have just left in y:
    rows outside the rank's range are zero and are not read; see grace_moe.h."""
    T, k = topk_weight.shape
    d = y.shape[1]
    if state.dtype != torch.int32 or state.numel() < SHARE_STATE_INTS:
        raise ValueError(f"state must hold {SHARE_STATE_INTS} int32")
    if out is None:
        out = torch.empty((T, d), dtype=y.dtype, device=y.device)
    _check(load_library().grace_combine_share(_dp(y), _dp(perm_pos), _dp(topk_weight), T, k, d, _dtype_code(y), _dp(y_shared),
                                              _dp(state), _dp(out), _stream()))
    return out


def grace_mfma_sustained(random_operands: bool = True, lds_fed: bool = True) -> float:
    """Sustained bf16 MFMA TFLOP/s of the current device (see grace_moe.h)."""
    out = C.c_double()
    _check(load_library().grace_mfma_sustained(int(random_operands), int(lds_fed), C.byref(out), _stream()))
    return float(out.value)


FFN_KERNELS = ("stream", "mid", "persist", "generic", "vector_f32")      # grace_kernel


def grace_ffn_kernel(up: bool, T: int, d: int, f: int, dt: int = GRACE_BF16, *, k: int = 1, S: int = 1, I: int = 1,
                     n_shared: int = 0, n_cu: int = 0) -> Tuple[str, int]:
    """(kernel, work-items) of a projection's launch (see grace_moe.h); with n_cu no device is needed."""
    kernel, items = C.c_int32(), C.c_int64()
    _check(load_library().grace_ffn_kernel(int(up), T, k, d, f, n_shared, S, I, dt, n_cu, C.byref(kernel), C.byref(items)))
    return FFN_KERNELS[kernel.value], int(items.value)


def grace_ffn_carries_rows(T: int, d: int, f: int, dt: int = GRACE_BF16, *, k: int = 1, S: int = 1, I: int = 1, n_shared: int = 0,
                           n_cu: int = 0) -> bool:
    """Does the gate+up projection's launch move the dispatch rows too (see grace_moe.h)?"""
    carried = C.c_int32()
    _check(load_library().grace_ffn_carries_rows(T, k, d, f, n_shared, S, I, dt, n_cu, C.byref(carried)))
    return bool(carried.value)
