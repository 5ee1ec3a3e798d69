"""Python binding of libsfc.so (C ABI in include/sfc.h): argument marshalling only.

Every step of the path runs in the library's HIP kernels; PyTorch supplies device memory and
streams.  There is no CPU fallback: importing works anywhere the shared library loads, but
every call needs a GPU, and a missing library is an error, not a reason to compute elsewhere.

The module-level functions carry the names of the C entry points and take torch tensors (device
tensors for d_* arguments).  `Cache` is a convenience holder for one cache, its output buffers
and its streams.
"""
from __future__ import annotations

import ctypes
import os
from typing import Optional

import numpy as np
import torch

_HERE = os.path.dirname(os.path.abspath(__file__))
LIB_PATH = os.path.join(_HERE, "libsfc.so")

SFC_OK, SFC_EINVAL, SFC_ESTATE, SFC_EHIP, SFC_ENOMEM, SFC_ELIMIT, SFC_ECORRUPT = 0, -1, -2, -3, -4, -5, -6
SFC_POLICY_LRU_BATCH = 0
SFC_POLICY_PREFETCH = 1
SFC_INDEX_AUTO, SFC_INDEX_HASHED, SFC_INDEX_DENSE = 0, 1, 2

EXPORTS = [
    "sfc_host_alloc", "sfc_host_free", "sfc_cache_create", "sfc_cache_destroy", "sfc_prepare",
    "sfc_fetch_misses", "sfc_lookup", "sfc_segment_sum", "sfc_backward_update", "sfc_flush",
    "sfc_get_stats", "sfc_cache_state", "sfc_profile_enable", "sfc_profile_read", "sfc_strerror",
    "sfc_last_error", "sfc_check", "sfc_peek_stats", "sfc_discard", "sfc_verify",
    "sfc_segment_sum_static",
]


class SfcError(RuntimeError):
    def __init__(self, code, msg):
        super().__init__("sfc error %d (%s): %s" % (code, _strerror(code), msg))
        self.code = code


class sfc_config(ctypes.Structure):
    _fields_ = [
        ("capacity_rows", ctypes.c_int64), ("dim", ctypes.c_int32), ("policy", ctypes.c_int32),
        ("max_ids_per_batch", ctypes.c_int64), ("max_bags_per_batch", ctypes.c_int64),
        ("host_rows", ctypes.c_int64), ("h_weights", ctypes.c_void_p), ("h_acc", ctypes.c_void_p),
        ("host_row_stride", ctypes.c_int64), ("lr", ctypes.c_float), ("eps", ctypes.c_float), ("lookahead", ctypes.c_int32),
        ("max_steps", ctypes.c_int32), ("stream", ctypes.c_void_p), ("side_stream", ctypes.c_void_p),
        ("optimizer", ctypes.c_int32), ("index_kind", ctypes.c_int32), ("host_state_stride", ctypes.c_int64),
        ("beta1", ctypes.c_double), ("beta2", ctypes.c_double),
    ]


class sfc_stats(ctypes.Structure):
    _fields_ = [(n, ctypes.c_int64) for n in
                ("n_unique", "n_hit", "n_miss", "n_evict", "n_bypass", "n_invalid", "h2d_bytes",
                 "d2h_bytes", "n_bad_offsets")]


def _load(path=None):
    path = path or LIB_PATH
    if not os.path.exists(path):
        raise RuntimeError(
            "libsfc.so is not built (%s); run `python paper_2104_08542_amd/build.py` or "
            "__graft_entry__.build(). There is no fallback path." % path)
    lib = ctypes.CDLL(path)
    vp, i64, i32, ci = ctypes.c_void_p, ctypes.c_int64, ctypes.c_int32, ctypes.c_int
    lib.sfc_host_alloc.restype, lib.sfc_host_alloc.argtypes = vp, [i64]
    lib.sfc_host_free.restype, lib.sfc_host_free.argtypes = None, [vp]
    lib.sfc_cache_create.restype = ci
    lib.sfc_cache_create.argtypes = [ctypes.POINTER(sfc_config), ctypes.POINTER(vp)]
    lib.sfc_cache_destroy.restype, lib.sfc_cache_destroy.argtypes = None, [vp]
    lib.sfc_prepare.restype, lib.sfc_prepare.argtypes = ci, [vp, vp, i64, vp, i64, vp, vp, vp, vp]
    lib.sfc_fetch_misses.restype, lib.sfc_fetch_misses.argtypes = ci, [vp]
    lib.sfc_lookup.restype, lib.sfc_lookup.argtypes = ci, [vp, vp]
    lib.sfc_segment_sum.restype, lib.sfc_segment_sum.argtypes = ci, [vp, vp, vp]
    lib.sfc_segment_sum_static.restype, lib.sfc_segment_sum_static.argtypes = ci, [vp, vp, vp]
    lib.sfc_backward_update.restype, lib.sfc_backward_update.argtypes = ci, [vp, vp]
    lib.sfc_flush.restype, lib.sfc_flush.argtypes = ci, [vp]
    lib.sfc_get_stats.restype, lib.sfc_get_stats.argtypes = ci, [vp, ctypes.POINTER(sfc_stats)]
    lib.sfc_cache_state.restype, lib.sfc_cache_state.argtypes = ci, [vp, vp, vp, vp, vp]
    lib.sfc_profile_enable.restype, lib.sfc_profile_enable.argtypes = ci, [vp, i32]
    lib.sfc_profile_read.restype = ci
    lib.sfc_profile_read.argtypes = [vp, i32, ctypes.POINTER(ctypes.c_double), ctypes.POINTER(i64)]
    lib.sfc_check.restype, lib.sfc_check.argtypes = ci, [vp]
    lib.sfc_peek_stats.restype = ci
    lib.sfc_peek_stats.argtypes = [vp, ctypes.POINTER(sfc_stats), ctypes.POINTER(i64)]
    lib.sfc_discard.restype, lib.sfc_discard.argtypes = ci, [vp]
    lib.sfc_verify.restype, lib.sfc_verify.argtypes = ci, [vp, ctypes.POINTER(i64)]
    lib.sfc_strerror.restype, lib.sfc_strerror.argtypes = ctypes.c_char_p, [ci]
    lib.sfc_last_error.restype, lib.sfc_last_error.argtypes = ctypes.c_char_p, []
    return lib


_lib = _load()
_I64, _I32, _F32 = torch.int64, torch.int32, torch.float32


def _strerror(code):
    return _lib.sfc_strerror(code).decode()


def _check(rc):
    if rc != SFC_OK:
        raise SfcError(rc, _lib.sfc_last_error().decode())


# The four calls of a step below: the marshalling is what a small batch waits for (32 x 39 ids looked up: 13.8 us of host
# time a pass, 9.4 of them in the library), so handles and addresses go to ctypes as plain integers, which its argument types take as they
# are, and a status is looked at before a function is called for it.
def _dptr(t: Optional[torch.Tensor], dtype=None):
    if t is None:
        return None
    if not t.is_cuda or not t.is_contiguous():
        raise ValueError("expected a contiguous device tensor")
    if dtype is not None and t.dtype is not dtype:
        raise ValueError("expected dtype %s, got %s" % (dtype, t.dtype))
    return t.data_ptr()


# ------------------------------------------------------------------ C entry points, same names

def sfc_host_alloc(nbytes: int) -> int:
    p = _lib.sfc_host_alloc(int(nbytes))
    if not p:
        raise SfcError(SFC_ENOMEM, "sfc_host_alloc(%d) failed" % nbytes)
    return p


def sfc_host_free(ptr: int) -> None:
    _lib.sfc_host_free(ctypes.c_void_p(ptr))


def sfc_cache_create(cfg: sfc_config) -> int:
    h = ctypes.c_void_p()
    _check(_lib.sfc_cache_create(ctypes.byref(cfg), ctypes.byref(h)))
    return h.value


def sfc_cache_destroy(h: int) -> None:
    _lib.sfc_cache_destroy(ctypes.c_void_p(h))


def sfc_prepare(h, d_ids, n_ids, d_offsets, n_bags, d_unique_ids, d_inverse, d_slot, d_miss_vids):
    rc = _lib.sfc_prepare(h, _dptr(d_ids, _I64), int(n_ids), _dptr(d_offsets, _I64), int(n_bags), _dptr(d_unique_ids, _I64),
                          _dptr(d_inverse, _I32), _dptr(d_slot, _I32), _dptr(d_miss_vids, _I32))
    if rc:
        _check(rc)


def sfc_fetch_misses(h):
    rc = _lib.sfc_fetch_misses(h)
    if rc:
        _check(rc)


def sfc_lookup(h, d_out):
    rc = _lib.sfc_lookup(h, _dptr(d_out, _F32))
    if rc:
        _check(rc)


def sfc_segment_sum(h, d_grad, d_common_grad):
    _check(_lib.sfc_segment_sum(ctypes.c_void_p(h), _dptr(d_grad, torch.float32),
                                _dptr(d_common_grad, torch.float32)))


def sfc_segment_sum_static(h, d_grad, d_common_grad):
    _check(_lib.sfc_segment_sum_static(ctypes.c_void_p(h), _dptr(d_grad, torch.float32),
                                       _dptr(d_common_grad, torch.float32)))


def sfc_backward_update(h, d_grad):
    rc = _lib.sfc_backward_update(h, _dptr(d_grad, _F32))
    if rc:
        _check(rc)


def sfc_flush(h):
    _check(_lib.sfc_flush(ctypes.c_void_p(h)))


def sfc_get_stats(h) -> dict:
    st = sfc_stats()
    _check(_lib.sfc_get_stats(ctypes.c_void_p(h), ctypes.byref(st)))
    return {k: int(getattr(st, k)) for k, _ in sfc_stats._fields_}


def sfc_check(h) -> None:
    """Raises SfcError if the device has reported an inconsistency or malformed offsets; never waits."""
    _check(_lib.sfc_check(ctypes.c_void_p(h)))


def sfc_peek_stats(h):
    """(stats dict, step) of the latest step the device has planned; never waits.  step 0: none yet."""
    st, step = sfc_stats(), ctypes.c_int64()
    _check(_lib.sfc_peek_stats(ctypes.c_void_p(h), ctypes.byref(st), ctypes.byref(step)))
    return {k: int(getattr(st, k)) for k, _ in sfc_stats._fields_}, step.value


def sfc_discard(h) -> None:
    rc = _lib.sfc_discard(h)
    if rc:
        _check(rc)


def sfc_verify(h):
    """Recount of the manager state on the device (test aid, synchronises): the four violation
    counts of include/sfc.h; raises SfcError(SFC_ECORRUPT) if any is nonzero."""
    bad = (ctypes.c_int64 * 4)()
    _check(_lib.sfc_verify(ctypes.c_void_p(h), bad))
    return list(bad)


def sfc_cache_state(h, capacity_rows, dim, rows=False, state_dim=None):
    """(slot_id[C] int64, stamp[C] int32[, rows[C,D], state[C,S]]) as numpy arrays."""
    sid = np.empty(capacity_rows, np.int64)
    stp = np.empty(capacity_rows, np.int32)
    w = np.empty((capacity_rows, dim), np.float32) if rows else None
    a = np.empty((capacity_rows, state_dim or dim), np.float32) if rows else None
    p = lambda x: None if x is None else x.ctypes.data_as(ctypes.c_void_p)
    _check(_lib.sfc_cache_state(ctypes.c_void_p(h), p(sid), p(stp), p(w), p(a)))
    return (sid, stp, w, a) if rows else (sid, stp)


def sfc_profile_enable(h, level: int):
    _check(_lib.sfc_profile_enable(ctypes.c_void_p(h), int(level)))


PROFILE_CALLS = ("prepare", "fetch_misses", "lookup", "backward_update", "k_seg_stream",
                 "k_seg_finish", "k_adagrad_rows")


def sfc_profile_read(h) -> dict:
    out = {}
    for i, name in enumerate(PROFILE_CALLS):
        ms, n = ctypes.c_double(), ctypes.c_int64()
        _check(_lib.sfc_profile_read(ctypes.c_void_p(h), i, ctypes.byref(ms), ctypes.byref(n)))
        out[name] = (ms.value, n.value)
    return out


# ------------------------------------------------------------------ conveniences

OPTIMIZERS = ("adagrad", "adam", "rowwise_adagrad")      # index = SFC_OPT_*


def state_floats(optimizer: str, dim: int) -> int:
    """S: floats of optimizer state that travel with one row."""
    return {"adagrad": dim, "adam": 2 * dim, "rowwise_adagrad": 4}[optimizer]


class HostTable:
    """[V, D] fp32 weights and [V, S] optimizer state in pinned, device-mapped host memory
    (S = state_floats(optimizer, D)).

    interleaved=True (default) stores row i as [weights_i | state_i] in one allocation, so a row's
    weights and optimizer state are one contiguous block for the host link; `w` and `acc` are then
    strided numpy views.  interleaved=False uses two separate contiguous arrays.
    """

    def __init__(self, rows: int, dim: int, interleaved: bool = True, optimizer: str = "adagrad",
                 align_floats: int = 1):
        self.rows, self.dim, self.interleaved = int(rows), int(dim), bool(interleaved)
        self.optimizer = optimizer
        S = self.state_dim = state_floats(optimizer, self.dim)
        if self.interleaved:
            # align_floats > 1 pads each [weights | state] block to a multiple of that many floats
            st = -(-(self.dim + S) // align_floats) * align_floats
            tot = self.rows * st
            self._base = sfc_host_alloc(tot * 4)
            self._pw, self._pa = self._base, self._base + 4 * self.dim
            self.stride = self.state_stride = st
            both = np.ctypeslib.as_array((ctypes.c_float * tot).from_address(self._base)
                                         ).reshape(self.rows, st)
            self.w, self.acc = both[:, :self.dim], both[:, self.dim:self.dim + S]
            self._bases = [self._base]
        else:
            self._pw = sfc_host_alloc(self.rows * self.dim * 4)
            try:
                self._pa = sfc_host_alloc(self.rows * S * 4)
            except SfcError:
                sfc_host_free(self._pw)
                raise
            self.stride, self.state_stride = self.dim, S
            mk = lambda p, k: np.ctypeslib.as_array((ctypes.c_float * (self.rows * k)).from_address(p)
                                                    ).reshape(self.rows, k)
            self.w, self.acc = mk(self._pw, self.dim), mk(self._pa, S)
            self._bases = [self._pw, self._pa]
        self.w_t, self.acc_t = torch.from_numpy(self.w), torch.from_numpy(self.acc)

    def free(self):
        if self._bases:
            self.w = self.acc = self.w_t = self.acc_t = None
            for b in self._bases:
                sfc_host_free(b)
            self._bases = []
            self._pw = self._pa = 0

    def __del__(self):
        try:
            self.free()
        except Exception:
            pass


class StepBuffers:
    """Device buffers of one prepared step (the d_* outputs of sfc_prepare) and its sizes."""

    def __init__(self, n, device):
        self.unique_ids = torch.empty(n, dtype=torch.int64, device=device)
        self.inverse = torch.empty(n, dtype=torch.int32, device=device)
        self.slot = torch.empty(n, dtype=torch.int32, device=device)
        self.miss_vids = torch.empty(n, dtype=torch.int32, device=device)
        self.n_ids = self.n_bags = 0
        self.keep = None          # the caller's ids / offsets stay alive as long as the step does


class Cache:
    """One sfc_cache with its output buffers; methods mirror the C calls of a step.

    lookahead = 0: prepare, fetch_misses, lookup, backward_update in that order.
    lookahead = L (1 .. 3): prepare / fetch_misses of step t+L may be issued before backward_update
    of step t (they run on other streams meanwhile); lookup and backward_update always act on the
    oldest step that has not been updated.  lookahead + 1 sets of output buffers rotate.
    """

    def __init__(self, table: HostTable, capacity_rows: int, max_ids: int, max_bags: Optional[int] = None,
                 lr=0.01, eps=1e-8, lookahead=0, max_steps=0, device="cuda:0", side_stream=True,
                 betas=(0.9, 0.999), policy=None, index_kind=SFC_INDEX_AUTO):
        self.table, self.C, self.D = table, int(capacity_rows), table.dim
        self.device = torch.device(device)
        self.max_ids = int(max_ids)
        self.max_bags = int(max_bags if max_bags is not None else max_ids)
        self.lookahead = int(lookahead)
        with torch.cuda.device(self.device):
            self.stream = torch.cuda.current_stream()
            self.side = torch.cuda.Stream() if (side_stream or lookahead) else self.stream
            cfg = sfc_config(self.C, self.D, SFC_POLICY_LRU_BATCH if policy is None else policy, self.max_ids, self.max_bags,
                             table.rows, table._pw, table._pa, table.stride, lr, eps, lookahead,
                             max_steps, self.stream.cuda_stream, self.side.cuda_stream,
                             OPTIMIZERS.index(table.optimizer), index_kind, table.state_stride,
                             betas[0], betas[1])
            self.h = sfc_cache_create(cfg)
            self.bufs = [StepBuffers(max(self.max_ids, 1), self.device) for _ in range(self.lookahead + 1)]
        self._next = 0
        self.last = self.bufs[0]        # most recently prepared step
        self.inflight = []              # prepared and not yet updated, oldest first

    def close(self):
        if getattr(self, "h", None):
            sfc_cache_destroy(self.h)
            self.h = None

    def __del__(self):
        try:
            self.close()
        except Exception:
            pass

    # outputs of the most recent prepare
    unique_ids = property(lambda self: self.last.unique_ids)
    inverse = property(lambda self: self.last.inverse)
    slot = property(lambda self: self.last.slot)
    miss_vids = property(lambda self: self.last.miss_vids)
    n_ids = property(lambda self: self.last.n_ids)
    n_bags = property(lambda self: self.last.n_bags)

    def prepare(self, ids: torch.Tensor, offsets: Optional[torch.Tensor] = None) -> StepBuffers:
        b = self.bufs[self._next]
        if self.inflight and b in self.inflight:            # rotation order broken by a discard: any set not in flight
            free = [x for x in self.bufs if x not in self.inflight]
            if free:
                b = free[0]
        n_ids = ids.numel()
        n_bags = n_ids if offsets is None else offsets.numel() - 1
        sfc_prepare(self.h, ids, n_ids, offsets, n_bags, b.unique_ids, b.inverse, b.slot, b.miss_vids)
        b.n_ids, b.n_bags, b.keep = n_ids, n_bags, (ids, offsets)
        self.inflight.append(b)
        self.last = b
        self._next = (self.bufs.index(b) + 1) % len(self.bufs)
        return b

    def fetch_misses(self):
        sfc_fetch_misses(self.h)

    def _current(self) -> StepBuffers:
        return self.inflight[0] if self.inflight else self.last

    def lookup(self, out: Optional[torch.Tensor] = None) -> torch.Tensor:
        b = self._current()
        if out is None:
            out = torch.empty(b.n_bags, self.D, dtype=torch.float32, device=self.device)
        sfc_lookup(self.h, out)
        return out

    def segment_sum(self, grad: torch.Tensor, out: Optional[torch.Tensor] = None) -> torch.Tensor:
        b = self._current()
        if out is None:
            out = torch.empty(max(b.n_ids, 1), self.D, dtype=torch.float32, device=self.device)
        sfc_segment_sum(self.h, grad, out)
        return out

    def backward_update(self, grad: torch.Tensor):
        sfc_backward_update(self.h, grad)
        if self.inflight:
            self.inflight.pop(0)

    def discard(self):
        """Give up the oldest fetched step without updating it (its rows stay cached)."""
        sfc_discard(self.h)
        if self.inflight:
            self.inflight.pop(0)

    def check(self):
        sfc_check(self.h)

    def peek_stats(self):
        return sfc_peek_stats(self.h)

    def verify(self):
        return sfc_verify(self.h)

    def flush(self):
        sfc_flush(self.h)

    def stats(self) -> dict:
        return sfc_get_stats(self.h)

    def state(self, rows=False):
        return sfc_cache_state(self.h, self.C, self.D, rows, self.table.state_dim)

    def step(self, ids, grad, offsets=None, out=None):
        self.prepare(ids, offsets)
        self.fetch_misses()
        out = self.lookup(out)
        self.backward_update(grad)
        return out
