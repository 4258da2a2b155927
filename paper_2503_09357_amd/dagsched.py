"""Thin Python binding of the C-ABI in include/dagsched.h (argument marshalling only).

Every step of the evaluation runs in the HIP kernels of ``libdagsched.so``; PyTorch is used for
device buffers and streams.  There is no CPU fallback: if the library cannot be loaded, or a
call fails, an exception is raised.
"""
from __future__ import annotations

import ctypes
from typing import Optional, Tuple

import numpy as np

from . import _build

OK, EINVAL, ECYCLE, EOVERFLOW, ENOMEM, EHIP, ESCRATCH = 0, -1, -2, -3, -4, -5, -6
STATIC_MAX_NODES = 32768
FLAG_OK, FLAG_CYCLIC, FLAG_BAD_PLACEMENT, FLAG_BAD_RANK, FLAG_INTERNAL, FLAG_OVER_MEMORY, FLAG_NO_CHANNEL = 0, 1, 2, 4, 8, 16, 32
NO_CHANNEL = -1      # off-diagonal comm entry of a machine pair without a channel (eq. (10))
CAND_MAJOR, CAND_MINOR = 0, 1
MAX_DEVICES, MAX_NODES = 64, 65535

EXPORTS = ("dagsched_validate", "dagsched_create", "dagsched_evaluate", "dagsched_evaluate_contended", "dagsched_destroy",
           "dagsched_strerror", "dagsched_get_info", "dagsched_plan", "dagsched_last_fallbacks", "dagsched_contended_info", "dagsched_time_evaluate", "dagsched_propose",
           "dagsched_propose_orders", "dagsched_select", "dagsched_schedule", "dagsched_schedule_static", "dagsched_coarsen")


class Desc(ctypes.Structure):
    _fields_ = [("n_nodes", ctypes.c_int32), ("n_edges", ctypes.c_int32), ("n_devices", ctypes.c_int32),
                ("row_ptr", ctypes.c_void_p), ("col_idx", ctypes.c_void_p), ("dur", ctypes.c_void_p),
                ("comm", ctypes.c_void_p), ("mem_delta", ctypes.c_void_p),
                ("max_candidates", ctypes.c_int32), ("layout", ctypes.c_int32), ("hip_device", ctypes.c_int32),
                ("weight", ctypes.c_void_p), ("mem_limit", ctypes.c_void_p), ("shape", ctypes.c_void_p),
                ("shared_placement", ctypes.c_void_p), ("contention", ctypes.c_int32)]


class Shape(ctypes.Structure):
    """dagsched_shape_t: optional launch shape of the evaluation kernels (0 / -1: chosen by the library)."""
    _fields_ = [("cand_per_block", ctypes.c_int32), ("ring_slots", ctypes.c_int32), ("feeders", ctypes.c_int32),
                ("placement_mode", ctypes.c_int32), ("block_threads", ctypes.c_int32), ("state_bits", ctypes.c_int32),
                ("preds_per_op", ctypes.c_int32), ("kernel", ctypes.c_int32), ("static_waves", ctypes.c_int32),
                ("ignore_shared_placement", ctypes.c_int32), ("window_cells", ctypes.c_int32)]


SHAPE_FIELDS = tuple(name for name, _ in Shape._fields_)

# Shape fields that every evaluator made inside a `shape_defaults` block starts from (an explicit `shape=` wins field
# by field).  For tests and tuning sweeps, which make evaluators in many places; empty otherwise.
_shape_defaults: dict = {}


class shape_defaults:
    """with shape_defaults(feeders=2, ring_slots=8): ...   (nests; restores the previous defaults on exit)"""

    def __init__(self, **fields):
        unknown = set(fields) - set(SHAPE_FIELDS)
        if unknown:
            raise ValueError("unknown shape fields: %s" % sorted(unknown))
        self.fields = fields

    def __enter__(self):
        global _shape_defaults
        self.old = _shape_defaults
        _shape_defaults = dict(_shape_defaults, **self.fields)
        return self

    def __exit__(self, *exc):
        global _shape_defaults
        _shape_defaults = self.old


class Info(ctypes.Structure):
    _fields_ = [("variant", ctypes.c_int32), ("cand_per_block", ctypes.c_int32), ("block_threads", ctypes.c_int32),
                ("lds_bytes", ctypes.c_int32), ("state_bits", ctypes.c_int32),
                ("ring_slots", ctypes.c_int16), ("kernel_kind", ctypes.c_int8), ("wide_ops", ctypes.c_int8),
                ("time_scale", ctypes.c_int32),
                ("feeders", ctypes.c_int8), ("placement_mode", ctypes.c_int8), ("preds_per_op", ctypes.c_int8),
                ("window_log2", ctypes.c_int8)]


class ContendedInfo(ctypes.Structure):
    _fields_ = [(k, ctypes.c_int32) for k in ("cand_per_block", "lanes_per_machine", "ring_slots", "block_threads", "ingest_teams", "left_over")]


class CoarsenParams(ctypes.Structure):
    _fields_ = [("target_nodes", ctypes.c_int32), ("edge_dur_max", ctypes.c_int64), ("edge_mem_max", ctypes.c_int64),
                ("nonedge_dur_max", ctypes.c_int64), ("nonedge_mem_max", ctypes.c_int64)]


class CoarsenResult(ctypes.Structure):
    _fields_ = [("n_coarse", ctypes.c_int32), ("n_coarse_edges", ctypes.c_int32), ("merges_edge", ctypes.c_int32),
                ("merges_nonedge", ctypes.c_int32)]


class DagschedError(RuntimeError):
    def __init__(self, code: int, text: str):
        super().__init__("dagsched error %d: %s" % (code, text))
        self.code = code


_lib = None


def load(import_torch_first: bool = True):
    """dlopen libdagsched.so (built in-tree).  PyTorch is imported first so that the library binds
    to the HIP runtime already resident in the process (one runtime, shared streams)."""
    global _lib
    if _lib is not None:
        return _lib
    if import_torch_first:
        import torch  # noqa: F401
    path = _build.ensure_hip()
    lib = ctypes.CDLL(path)
    vp, i32 = ctypes.c_void_p, ctypes.c_int32
    lib.dagsched_validate.restype = ctypes.c_int
    lib.dagsched_validate.argtypes = [ctypes.POINTER(Desc)]
    lib.dagsched_create.restype = ctypes.c_int
    lib.dagsched_create.argtypes = [ctypes.POINTER(Desc), ctypes.POINTER(vp)]
    lib.dagsched_evaluate.restype = ctypes.c_int
    lib.dagsched_evaluate.argtypes = [vp, i32, vp, vp, vp, vp, vp, vp, vp]
    lib.dagsched_evaluate_contended.restype = ctypes.c_int
    lib.dagsched_evaluate_contended.argtypes = [vp, i32, vp, vp, vp, vp, vp, vp, vp, vp]
    lib.dagsched_time_evaluate.restype = ctypes.c_int
    lib.dagsched_time_evaluate.argtypes = [vp, i32, vp, vp, vp, vp, vp, vp, vp, i32, ctypes.POINTER(ctypes.c_float)]
    lib.dagsched_destroy.restype = None
    lib.dagsched_destroy.argtypes = [vp]
    lib.dagsched_strerror.restype = ctypes.c_char_p
    lib.dagsched_strerror.argtypes = [ctypes.c_int]
    lib.dagsched_get_info.restype = ctypes.c_int
    lib.dagsched_get_info.argtypes = [vp, ctypes.POINTER(Info)]
    lib.dagsched_plan.restype = ctypes.c_int
    lib.dagsched_plan.argtypes = [ctypes.POINTER(Desc), i32, i32, ctypes.POINTER(Info)]
    lib.dagsched_last_fallbacks.restype = ctypes.c_int
    lib.dagsched_last_fallbacks.argtypes = [vp, vp, ctypes.POINTER(ctypes.c_int32)]
    lib.dagsched_contended_info.restype = ctypes.c_int
    lib.dagsched_contended_info.argtypes = [vp, vp, ctypes.POINTER(ContendedInfo)]
    lib.dagsched_propose.restype = ctypes.c_int
    lib.dagsched_propose.argtypes = [vp, i32, vp, vp, vp, vp, vp, vp]
    lib.dagsched_propose_orders.restype = ctypes.c_int
    lib.dagsched_propose_orders.argtypes = [vp, i32, vp, vp, vp, vp, vp, vp]
    lib.dagsched_select.restype = ctypes.c_int
    lib.dagsched_select.argtypes = [vp, i32, vp, vp, vp, vp]
    lib.dagsched_schedule.restype = ctypes.c_int
    lib.dagsched_schedule.argtypes = [vp, vp, vp, vp, vp, vp, vp]
    lib.dagsched_schedule_static.restype = ctypes.c_int
    lib.dagsched_schedule_static.argtypes = [vp, vp, vp, vp, vp, vp, vp]
    lib.dagsched_coarsen.restype = ctypes.c_int
    lib.dagsched_coarsen.argtypes = [i32, i32, vp, vp, vp, vp, vp, ctypes.POINTER(CoarsenParams), i32, vp, vp, vp, vp, vp, vp,
                                     ctypes.POINTER(CoarsenResult)]
    _lib = lib
    return lib


def strerror(code: int) -> str:
    return load().dagsched_strerror(code).decode()


def _check(code: int):
    if code != OK:
        raise DagschedError(code, strerror(code))


NO_MERGES, NO_LIMIT = -1, 2 ** 62     # thresholds of coarsen: that kind of merge off / no bound


def coarsen(row_ptr, col_idx, dur, mem_delta, mem_req=None, target=1, edge_dur_max=NO_LIMIT, edge_mem_max=NO_LIMIT,
            nonedge_dur_max=NO_LIMIT, nonedge_mem_max=NO_LIMIT, hip_device: int = 0) -> dict:
    """dagsched_coarsen (Sec. IV, Alg. 1) on host arrays -> dict(n_coarse, node_map [N], row_ptr, col_idx, dur,
    mem_delta, mem_req, merges_edge, merges_nonedge) of the coarse graph."""
    rp = np.ascontiguousarray(row_ptr, dtype=np.int32)
    ci = np.ascontiguousarray(col_idx, dtype=np.int32)
    n, e = len(rp) - 1, len(ci)
    d = np.ascontiguousarray(dur, dtype=np.int32)
    m = np.ascontiguousarray(mem_delta, dtype=np.int64)
    r = None if mem_req is None else np.ascontiguousarray(mem_req, dtype=np.int64)
    if d.shape != (n,) or m.shape != (n,) or (r is not None and r.shape != (n,)):
        raise ValueError("dur, mem_delta and mem_req must have one entry per node")
    params = CoarsenParams(int(target), int(edge_dur_max), int(edge_mem_max), int(nonedge_dur_max), int(nonedge_mem_max))
    res = CoarsenResult()
    node_map = np.empty(max(n, 1), np.int32)
    c_rp, c_ci = np.empty(max(n, 0) + 1, np.int32), np.empty(max(e, 1), np.int32)
    c_d, c_m, c_r = np.empty(max(n, 1), np.int32), np.empty(max(n, 1), np.int64), np.empty(max(n, 1), np.int64)
    ptr = lambda a: a.ctypes.data if a is not None and a.size else None
    _check(load().dagsched_coarsen(n, e, ptr(rp), ptr(ci), ptr(d), ptr(m), ptr(r), ctypes.byref(params), hip_device,
                                   ptr(node_map), ptr(c_rp), ptr(c_ci), ptr(c_d), ptr(c_m), ptr(c_r), ctypes.byref(res)))
    k = res.n_coarse
    return dict(n_coarse=k, node_map=node_map[:n].copy(), row_ptr=c_rp[:k + 1].copy(), col_idx=c_ci[:res.n_coarse_edges].copy(),
                dur=c_d[:k].copy(), mem_delta=c_m[:k].copy(), mem_req=c_r[:k].copy(), merges_edge=res.merges_edge,
                merges_nonedge=res.merges_nonedge)


class _HostProblem:
    """Keeps the contiguous host arrays alive while a Desc points at them."""

    def __init__(self, n_devices, row_ptr, col_idx, dur, comm, mem_delta, max_candidates, layout, hip_device,
                 n_nodes=None, n_edges=None, weight=None, mem_limit=None, shape=None, shared_placement=None,
                 contention=False):
        self.row_ptr = np.ascontiguousarray(row_ptr, dtype=np.int32)
        self.col_idx = np.ascontiguousarray(col_idx, dtype=np.int32)
        self.dur = np.ascontiguousarray(dur, dtype=np.int32)
        self.comm = np.ascontiguousarray(comm, dtype=np.int32).reshape(-1)
        self.mem_delta = np.ascontiguousarray(mem_delta, dtype=np.int64)
        d = Desc()
        d.n_nodes = len(self.row_ptr) - 1 if n_nodes is None else n_nodes
        d.n_edges = len(self.col_idx) if n_edges is None else n_edges
        d.n_devices = n_devices
        d.row_ptr = self.row_ptr.ctypes.data if self.row_ptr.size else None
        d.col_idx = self.col_idx.ctypes.data if self.col_idx.size else None
        d.dur = self.dur.ctypes.data if self.dur.size else None
        d.comm = self.comm.ctypes.data if self.comm.size else None
        d.mem_delta = self.mem_delta.ctypes.data if self.mem_delta.size else None
        d.max_candidates = max_candidates
        d.layout = layout
        d.hip_device = hip_device
        self.weight = None if weight is None else np.ascontiguousarray(weight, dtype=np.int64)
        self.mem_limit = None if mem_limit is None else np.ascontiguousarray(mem_limit, dtype=np.int64)
        if self.weight is not None and self.weight.shape != (d.n_nodes,):
            raise ValueError("weight must have one entry per node")
        if self.mem_limit is not None and self.mem_limit.shape != (n_devices,):
            raise ValueError("mem_limit must have one entry per machine")
        d.weight = None if self.weight is None else self.weight.ctypes.data
        d.mem_limit = None if self.mem_limit is None else self.mem_limit.ctypes.data
        self.shape = None
        if shape is not None or _shape_defaults:
            shape = dict(_shape_defaults, **(shape or {}))
            unknown = set(shape) - set(SHAPE_FIELDS)
            if unknown:
                raise ValueError("unknown shape fields: %s" % sorted(unknown))
            self.shape = Shape(*[int(shape.get(f, -1 if f == "placement_mode" else 0)) for f in SHAPE_FIELDS])
        d.shape = None if self.shape is None else ctypes.addressof(self.shape)
        self.shared_placement = None if shared_placement is None else np.ascontiguousarray(shared_placement, dtype=np.int32).reshape(-1)
        if self.shared_placement is not None and self.shared_placement.shape != (d.n_nodes,):
            raise ValueError("shared_placement must have one entry per node")
        d.shared_placement = None if self.shared_placement is None else self.shared_placement.ctypes.data
        d.contention = 1 if contention else 0
        self.desc = d


def validate(n_devices, row_ptr, col_idx, dur, comm, mem_delta, max_candidates=1, layout=CAND_MAJOR,
             n_nodes=None, n_edges=None, weight=None, mem_limit=None, shape=None, shared_placement=None,
             contention=False) -> int:
    """Host-only description check; returns the code dagsched_create would return."""
    hp = _HostProblem(n_devices, row_ptr, col_idx, dur, comm, mem_delta, max_candidates, layout, 0, n_nodes, n_edges,
                      weight, mem_limit, shape, shared_placement, contention)
    return load(import_torch_first=False).dagsched_validate(ctypes.byref(hp.desc))


def _info_dict(i: "Info") -> dict:
    d = {k: getattr(i, k) for k in ("variant", "cand_per_block", "block_threads", "lds_bytes", "state_bits",
                                    "ring_slots", "time_scale", "feeders", "preds_per_op", "kernel_kind", "wide_ops",
                                    "window_log2")}
    d.update(kernel_kind=i.kernel_kind & 3, two_launches=i.kernel_kind >> 2)
    d["placement_bytes_in_lds"] = i.placement_mode
    return d


def plan(n_devices, row_ptr, col_idx, dur, comm, mem_delta, max_candidates=1, layout=CAND_MAJOR, weight=None,
         mem_limit=None, shape=None, shared_placement=None, lds_bytes: int = 160 * 1024, n_cu: int = 256) -> dict:
    """Host-only: the kernel variant and shape dagsched_create would choose (dagsched_plan); raises on a bad description."""
    hp = _HostProblem(n_devices, row_ptr, col_idx, dur, comm, mem_delta, max_candidates, layout, 0, weight=weight,
                      mem_limit=mem_limit, shape=shape, shared_placement=shared_placement)
    i = Info()
    _check(load(import_torch_first=False).dagsched_plan(ctypes.byref(hp.desc), lds_bytes, n_cu, ctypes.byref(i)))
    return _info_dict(i)


class Evaluator:
    """dagsched_create / dagsched_evaluate / dagsched_destroy around torch device tensors."""

    def __init__(self, n_devices, row_ptr, col_idx, dur, comm, mem_delta, max_candidates: int,
                 layout: int = CAND_MAJOR, hip_device: int = 0, weight=None, mem_limit=None, shape=None,
                 shared_placement=None, contention: bool = False):
        """shared_placement: [N] machine of every operation when (nearly) all candidates will place alike and differ
        in the orders only; a hint that selects a faster kernel, never changes a result.
        contention: the handle will also be used for evaluate_contended (channel contention, eqs. (11)-(15))."""
        lib = load()
        hp = _HostProblem(n_devices, row_ptr, col_idx, dur, comm, mem_delta, max_candidates, layout, hip_device,
                          weight=weight, mem_limit=mem_limit, shape=shape, shared_placement=shared_placement,
                          contention=contention)
        handle = ctypes.c_void_p()
        _check(lib.dagsched_create(ctypes.byref(hp.desc), ctypes.byref(handle)))
        self._h = handle
        self.N, self.P, self.E = hp.desc.n_nodes, n_devices, hp.desc.n_edges
        self.layout, self.max_candidates, self.hip_device = layout, max_candidates, hip_device

    @classmethod
    def for_workload(cls, w, max_candidates: Optional[int] = None, layout: int = CAND_MAJOR, hip_device: int = 0,
                     shape=None, shared_placement="auto", contention: bool = False):
        """shared_placement "auto": pass the hint when the workload has several candidates and all place alike."""
        if isinstance(shared_placement, str):
            pl = np.asarray(w.placement)
            same = pl.shape[0] > 1 and bool((pl == pl[0]).all()) and bool(((pl[0] >= 0) & (pl[0] < w.n_devices)).all())
            shared_placement = pl[0] if same else None
        return cls(w.n_devices, w.row_ptr, w.col_idx, w.dur, w.comm, w.mem_delta,
                   w.n_cand if max_candidates is None else max_candidates, layout, hip_device,
                   weight=getattr(w, "weight", None), mem_limit=getattr(w, "mem_limit", None), shape=shape,
                   shared_placement=shared_placement, contention=contention)

    @classmethod
    def autotuned(cls, make, placement, rank, reps: int = 3, verbose: bool = False):
        """Time the library's own launch shape and a few neighbours of it (one feeder more or fewer, half the
        candidates per workgroup, the placement elsewhere) on the caller's batch and return the fastest evaluator
        with the shape it uses.  `make(shape)` builds an Evaluator for the caller's problem with a dagsched_shape_t
        given as a dict (None: the library's choice).  Shapes that the library answers with its int32 kernel are
        skipped.  Worth it when very many batches of one problem follow (a search)."""
        best = make(None)
        base = best.info()
        out = best.alloc_outputs(best._n_cand(placement, rank))
        best.evaluate(placement, rank, out)
        best_ms, best_shape = best.time_evaluate(placement, rank, out, reps=reps), None
        if base["variant"] not in (3, 4, 5):              # the int32 kernel has no shapes to choose from
            return best, best_shape
        trials = []
        for f in (base["feeders"] - 1, base["feeders"] + 1):
            if 1 <= f <= 4:
                trials.append({"feeders": f})
        if base["cand_per_block"] > 1:
            trials.append({"cand_per_block": base["cand_per_block"] // 2})
        trials += [{"placement_mode": m} for m in (0, 1, 2) if m != base["placement_bytes_in_lds"]]
        for shape in trials:
            try:
                ev = make(shape)
            except DagschedError:
                continue
            keep = False
            if ev.info()["variant"] in (3, 4, 5):
                ev.evaluate(placement, rank, out)
                ms = ev.time_evaluate(placement, rank, out, reps=reps)
                if verbose:
                    print("autotune", shape, "%.4f ms (best so far %.4f ms)" % (ms, best_ms))
                if ms < 0.97 * best_ms:                # a clear win only: timings of one batch are noisy
                    best.close()
                    best, best_ms, best_shape, keep = ev, ms, shape, True
            if not keep:
                ev.close()
        return best, best_shape

    def info(self) -> dict:
        i = Info()
        _check(load().dagsched_get_info(self._h, ctypes.byref(i)))
        return _info_dict(i)

    def last_fallbacks(self, stream=None) -> int:
        """Candidates of the last evaluate that another kernel evaluated again, or instead (synchronises the stream)."""
        import torch
        s = torch.cuda.current_stream(self.hip_device) if stream is None else stream
        n = ctypes.c_int32()
        _check(load().dagsched_last_fallbacks(self._h, s.cuda_stream, ctypes.byref(n)))
        return int(n.value)

    def contended_info(self, stream=None) -> dict:
        """Shape of the contended evaluation's fast path, and the candidates that the last evaluate_contended left to the
        general kernel (synchronises the stream)."""
        import torch
        s = torch.cuda.current_stream(self.hip_device) if stream is None else stream
        i = ContendedInfo()
        _check(load().dagsched_contended_info(self._h, s.cuda_stream, ctypes.byref(i)))
        return {k: getattr(i, k) for k, _ in ContendedInfo._fields_}

    def _n_cand(self, placement, rank) -> int:
        import torch
        for t in (placement, rank):
            if not (t.is_cuda and t.dtype == torch.int32 and t.is_contiguous() and t.dim() == 2):
                raise ValueError("placement/rank must be contiguous 2-D int32 device tensors")
        shape = tuple(placement.shape)
        if tuple(rank.shape) != shape:
            raise ValueError("placement and rank differ in shape")
        if self.layout == CAND_MAJOR:
            if shape[1] != self.N:
                raise ValueError("candidate-major tensors must be [C, N]")
            return shape[0]
        if shape[0] != self.N:
            raise ValueError("candidate-minor tensors must be [N, C]")
        return shape[1]

    def alloc_outputs(self, n_cand: int):
        import torch
        dev = torch.device("cuda", self.hip_device)
        pk_shape = (n_cand, self.P) if self.layout == CAND_MAJOR else (self.P, n_cand)
        return (torch.empty(n_cand, dtype=torch.int32, device=dev), torch.empty(n_cand, dtype=torch.int64, device=dev),
                torch.empty(pk_shape, dtype=torch.int64, device=dev), torch.empty(n_cand, dtype=torch.int32, device=dev))

    def evaluate(self, placement, rank, out: Optional[Tuple] = None, stream=None):
        """Enqueue one evaluation on ``stream`` (default: torch's current stream); asynchronous.
        Returns (makespan int32 [C], bubble int64 [C], peak_mem int64 [C,P] | [P,C], flags int32 [C])."""
        import torch
        n_cand = self._n_cand(placement, rank)
        if out is None:
            out = self.alloc_outputs(n_cand)
        z, b, pk, f = out
        s = torch.cuda.current_stream(self.hip_device) if stream is None else stream
        _check(load().dagsched_evaluate(self._h, n_cand, placement.data_ptr(), rank.data_ptr(), z.data_ptr(),
                                        b.data_ptr(), pk.data_ptr(), f.data_ptr(), s.cuda_stream))
        return out

    def evaluate_contended(self, placement, rank, edge_rank, out: Optional[Tuple] = None, stream=None):
        """Evaluation with channel contention: edge_rank is a device int32 tensor [C, E] (candidate-major) or [E, C],
        the rank of every DAG edge's transfer on its channel.  Same outputs as evaluate; asynchronous."""
        import torch
        n_cand = self._n_cand(placement, rank)
        want = (n_cand, self.E) if self.layout == CAND_MAJOR else (self.E, n_cand)
        if not (edge_rank.is_cuda and edge_rank.dtype == torch.int32 and edge_rank.is_contiguous() and tuple(edge_rank.shape) == want):
            raise ValueError("edge_rank must be a contiguous int32 device tensor of shape %s" % (want,))
        if out is None:
            out = self.alloc_outputs(n_cand)
        z, b, pk, f = out
        s = torch.cuda.current_stream(self.hip_device) if stream is None else stream
        _check(load().dagsched_evaluate_contended(self._h, n_cand, placement.data_ptr(), rank.data_ptr(),
                                                  edge_rank.data_ptr() if self.E else None, z.data_ptr(), b.data_ptr(),
                                                  pk.data_ptr(), f.data_ptr(), s.cuda_stream))
        return out

    def time_evaluate(self, placement, rank, out, reps: int, stream=None) -> float:
        """Mean milliseconds per evaluation over ``reps`` back-to-back launches (HIP events on the stream)."""
        import torch
        n_cand = self._n_cand(placement, rank)
        z, b, pk, f = out
        s = torch.cuda.current_stream(self.hip_device) if stream is None else stream
        ms = ctypes.c_float()
        _check(load().dagsched_time_evaluate(self._h, n_cand, placement.data_ptr(), rank.data_ptr(), z.data_ptr(),
                                             b.data_ptr(), pk.data_ptr(), f.data_ptr(), s.cuda_stream, reps,
                                             ctypes.byref(ms)))
        return float(ms.value)

    def propose(self, base_placement, base_rank, rnd, out: Optional[Tuple] = None, stream=None, orders_only: bool = False):
        """One-move neighbourhood of a base schedule (device int32 [N] each); ``rnd`` is a device tensor of
        4 * n_cand random 32-bit words (int32 or uint32 storage).  Returns (placement, rank) in the handle's
        layout; candidate 0 is the base.  orders_only: every candidate keeps the base's placement."""
        import torch
        n_cand = rnd.numel() // 4
        dev = torch.device("cuda", self.hip_device)
        if out is None:
            shape = (n_cand, self.N) if self.layout == CAND_MAJOR else (self.N, n_cand)
            out = (torch.empty(shape, dtype=torch.int32, device=dev), torch.empty(shape, dtype=torch.int32, device=dev))
        s = torch.cuda.current_stream(self.hip_device) if stream is None else stream
        call = load().dagsched_propose_orders if orders_only else load().dagsched_propose
        _check(call(self._h, n_cand, base_placement.data_ptr(), base_rank.data_ptr(), rnd.data_ptr(),
                    out[0].data_ptr(), out[1].data_ptr(), s.cuda_stream))
        return out

    def select(self, makespan, flags, out=None, stream=None):
        """Device int32 [2]: (index, makespan) of the best feasible candidate, (-1, -1) if there is none."""
        import torch
        if out is None:
            out = torch.empty(2, dtype=torch.int32, device=torch.device("cuda", self.hip_device))
        s = torch.cuda.current_stream(self.hip_device) if stream is None else stream
        _check(load().dagsched_select(self._h, makespan.numel(), makespan.data_ptr(), flags.data_ptr(), out.data_ptr(),
                                      s.cuda_stream))
        return out

    def schedule(self, placement, rank, stream=None, out=None, static_scratch: bool = False):
        """Start / end times of ONE candidate (device int32 [N] each) -> (start int32 [N], end int32 [N], flag int32 [1]).
        static_scratch: through dagsched_schedule_static, whose scratch is a static device array of the library."""
        import torch
        dev = torch.device("cuda", self.hip_device)
        if out is None:
            out = (torch.empty(self.N, dtype=torch.int32, device=dev), torch.empty(self.N, dtype=torch.int32, device=dev),
                   torch.empty(1, dtype=torch.int32, device=dev))
        start, end, flag = out
        s = torch.cuda.current_stream(self.hip_device) if stream is None else stream
        call = load().dagsched_schedule_static if static_scratch else load().dagsched_schedule
        _check(call(self._h, placement.data_ptr(), rank.data_ptr(), start.data_ptr(), end.data_ptr(), flag.data_ptr(),
                    s.cuda_stream))
        return start, end, flag

    def close(self):
        if self._h:
            load().dagsched_destroy(self._h)
            self._h = None

    def __enter__(self):
        return self

    def __exit__(self, *exc):
        self.close()

    def __del__(self):
        try:
            self.close()
        except Exception:
            pass
