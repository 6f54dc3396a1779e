"""MI355X (gfx950) maximum common induced subgraph search -- Python binding.

The search (McSplit branch and bound: class split by adjacency, Eq. 1 bound,
device work queue, atomic incumbents) runs in the HIP library libmcs.so behind
the C ABI of include/mcs.h.  This module only marshals arguments; PyTorch
supplies the device workspace and the stream.

Graphs are dicts {"n", "directed", "rows", "label"}: rows[i] is an int whose
bit j is set iff the arc i -> j exists; label is None or a list of n ints.
"""
from __future__ import annotations

import ctypes
import struct
from array import array
from dataclasses import dataclass, field

import numpy as np

from . import _abi

__all__ = ["McsError", "Plan", "solve", "solve_batch", "solve_goals", "workspace_size",
           "Tuning", "status_string"]


class McsError(RuntimeError):
    def __init__(self, status: int, detail: str):
        self.status = status
        super().__init__(f"{status_string(status)} ({status}): {detail}")


def status_string(s: int) -> str:
    return _abi.load().mcs_status_string(s).decode()


def _last_error() -> str:
    return _abi.load().mcs_last_error().decode()


@dataclass
class Tuning:
    waves_per_cu: int = 0
    children_per_wave: int = 0
    ring_slots: int = 0
    donate_low: int = 0
    donate_depth: int = 0
    check_interval: int = 0
    no_reprune: int = 0
    single_wave: int = 0
    use_graph: int = 0
    stack_classes: int = 0
    backoff_max: int = 0
    seg_lanes: int = 0

    def to_c(self) -> _abi.mcs_tuning:
        return _abi.mcs_tuning(self.waves_per_cu, self.children_per_wave, self.ring_slots,
                               self.donate_low, self.donate_depth, self.check_interval,
                               self.no_reprune, self.single_wave, self.use_graph,
                               self.stack_classes, self.backoff_max, self.seg_lanes)


_GRAPH = struct.Struct("@iiPP")      # mcs_graph
_RESULT = struct.Struct("@iiPPqdd")  # mcs_result
_MAP_AT = _abi.mcs_result.map_g.offset
_MAP_PTRS = struct.Struct("@PP")     # mcs_result.map_g, .map_h
_LABELS = (list, tuple, array, np.ndarray)


class _Marshal:
    """The mcs_graph arrays of a list of pairs, and the buffers behind them.

    All row words of the batch go into one buffer, the labels into another:
    a numpy array, its ctypes pointers and a Python loop over the rows of each
    graph took 72 ms for 4,096 pairs of 10 to 22 vertices, this and the
    plan's creation take 12.  Graphs that the flat form does not take as they
    are (more vertices than the library allows, rows with bits above their
    words, entries that are no integers, labels that may be gone through only
    once: _graph goes through them itself) go one by one through _graph, which
    converts or refuses them.
    """

    def __init__(self, pairs):
        n = len(pairs)
        self.G = (_abi.mcs_graph * max(n, 1))()
        self.H = (_abi.mcs_graph * max(n, 1))()
        self.sizes = []    # min(n(G), n(H)) per pair, at least 1
        self._flat = None  # (words, labels, their extents per graph)
        try:
            self._marshal_flat(pairs)
        except (TypeError, ValueError, OverflowError, DeprecationWarning):
            self._flat = None
            self.sizes = []
            self._keep = []
            for i, (g, h) in enumerate(pairs):
                self.G[i] = self._graph(g)
                self.H[i] = self._graph(h)
                self.sizes.append(max(1, min(self.G[i].n, self.H[i].n)))

    def _marshal_flat(self, pairs):
        words, labels, recs = array("Q"), array("i"), []
        for g, h in pairs:
            ns = []
            for x in (g, h):
                n = int(x["n"])
                if not 0 <= n <= _abi.MCS_MAX_N:
                    raise ValueError("general path")
                at = len(words)
                if n <= 64:
                    words.extend(x["rows"][:n])
                    end = at + max(n, 1)
                else:
                    # ceil(n / 64) words a row, the low one first
                    rb = 8 * ((n + 63) // 64)
                    words.frombytes(b"".join([int(r).to_bytes(rb, "little")
                                              for r in x["rows"][:n]]))
                    end = at + n * rb // 8
                if len(words) < end:
                    words.frombytes(bytes(8 * (end - len(words))))
                lab, lab_at = x.get("label"), -1
                if lab is not None:
                    if not isinstance(lab, _LABELS):
                        raise ValueError("general path")
                    lab_at = len(labels)
                    labels.extend(lab)
                    if len(labels) == lab_at:
                        labels.append(0)
                recs.append((n, 1 if x.get("directed") else 0, at, end, lab_at, len(labels)))
                ns.append(n)
            self.sizes.append(max(1, min(ns)))
        wp, lp = words.buffer_info()[0], labels.buffer_info()[0]
        put, size = _GRAPH.pack_into, _GRAPH.size
        for i, (n, directed, at, _, lab_at, _) in enumerate(recs):
            put(self.H if i & 1 else self.G, size * (i >> 1), n, directed, wp + 8 * at,
                lp + 4 * lab_at if lab_at >= 0 else 0)
        self._flat = (words, labels, recs)

    @property
    def keep(self):
        """The buffers behind the graphs, in order: each graph's row words,
        then its labels if it has any."""
        if self._flat is None:
            return self._keep
        words, labels, recs = self._flat
        out = []
        for _, _, at, end, lab_at, lab_end in recs:
            out.append(np.frombuffer(words, np.uint64)[at:end])
            if lab_at >= 0:
                out.append(np.frombuffer(labels, np.int32)[lab_at:lab_end])
        return out

    def _graph(self, g) -> _abi.mcs_graph:
        n = int(g["n"])
        # rw 64-bit words per row: one up to 64 vertices, ceil(n / 64) above
        rw = 1 if n <= 64 else (n + 63) // 64
        rows = np.zeros(max(n, 1) * rw, dtype=np.uint64)
        for i, r in enumerate(g["rows"][:max(n, 0)]):
            for k in range(rw):
                rows[i * rw + k] = np.uint64((int(r) >> (64 * k)) & 0xFFFFFFFFFFFFFFFF)
        self._keep.append(rows)
        lab = None
        if g.get("label") is not None:
            la = np.array(list(g["label"]) or [0], dtype=np.int32)
            self._keep.append(la)
            lab = la.ctypes.data_as(ctypes.POINTER(ctypes.c_int32))
        return _abi.mcs_graph(n, 1 if g.get("directed") else 0,
                              rows.ctypes.data_as(ctypes.POINTER(ctypes.c_uint64)), lab)


ORDERINGS = {"degree": 0, "btf": 1, "portfolio": 2}


def _opts(node_limit, time_limit_s, tuning, policy=None, policy_depth=0, policy_mode=0,
          ordering="degree", deadend_nodes=0, deadend_ratio=0):
    """policy: a torch half tensor of packed parameters on the device (or an
    object with .half_params, see policy.Policy).  ordering: "degree",
    "btf" or "portfolio" (both orders racing on one incumbent;
    mcs_opts.ordering)."""
    t = None
    tc = None
    if tuning is not None:
        tc = tuning.to_c() if isinstance(tuning, Tuning) else Tuning(**tuning).to_c()
        t = ctypes.pointer(tc)
    ptr = None
    if policy is not None:
        hp = getattr(policy, "half_params", policy)
        ptr = ctypes.c_void_p(hp.data_ptr())
    o = _abi.mcs_opts(int(node_limit or 0), float(time_limit_s or 0.0), t, ptr,
                      int(policy_depth), int(policy_mode), ORDERINGS[ordering],
                      int(deadend_ratio), int(deadend_nodes))
    return o, tc


def _torch():
    import torch
    if not torch.cuda.is_available():
        raise RuntimeError("no GPU visible: the search runs only on the HIP device")
    return torch


@dataclass
class Result:
    size: int
    optimal: bool
    mapping: list
    nodes: int
    t_best_s: float
    t_proof_s: float


class _Results:
    """An mcs_result array with room for every mapping in one buffer (sizes:
    the largest size of each pair), and the Result list made from it."""

    def __init__(self, sizes):
        self.res = (_abi.mcs_result * max(len(sizes), 1))()
        self.at = at = [0]
        for c in sizes:
            at.append(at[-1] + c)
        self.map_g = (ctypes.c_int32 * max(at[-1], 1))()
        self.map_h = (ctypes.c_int32 * max(at[-1], 1))()
        g, h = ctypes.addressof(self.map_g), ctypes.addressof(self.map_h)
        put, step = _MAP_PTRS.pack_into, _RESULT.size
        for i in range(len(sizes)):
            put(self.res, step * i + _MAP_AT, g + 4 * at[i], h + 4 * at[i])

    def results(self):
        mg, mh, out = self.map_g, self.map_h, []
        for a, (size, optimal, _, _, nodes, t_best, t_proof) in zip(
                self.at[:-1], _RESULT.iter_unpack(self.res)):
            b = a + max(size, 0)
            out.append(Result(size, bool(optimal), list(zip(mg[a:b], mh[a:b])), nodes, t_best,
                              t_proof))
        return out


@dataclass
class Stats:
    nodes: int = 0
    batches: int = 0
    children: int = 0
    lane_slots: int = 0
    donations: int = 0
    pops: int = 0
    waves: int = 0
    blocks: int = 0
    lds_per_wave: int = 0
    stopped: int = 0
    kernel_ms: float = 0.0
    busy_wave_s: float = 0.0
    hbm_frames: int = 0
    stack_classes: int = 0
    max_stack_used: int = 0
    sleep_wave_s: float = 0.0
    lds_bytes: int = 0
    node_classes: int = 0
    extra: dict = field(default_factory=dict)

    @property
    def busy_frac(self) -> float:
        """Share of the launch's wavefront-time spent searching."""
        span = self.waves * self.kernel_ms * 1e-3
        return self.busy_wave_s / span if span > 0 else 0.0


class Plan:
    """A batch of pairs prepared once (mcs_plan_create), uploaded once into a
    torch-allocated workspace (mcs_plan_upload), then run any number of times
    (mcs_plan_run) -- inputs stay resident in HBM between runs."""

    def __init__(self, pairs, node_limit=0, time_limit_s=0.0, tuning=None, policy=None,
                 policy_depth=1, policy_mode=0, ordering="degree", deadend_nodes=0,
                 deadend_ratio=0):
        self.lib = _abi.load()
        self.pairs = list(pairs)
        self._m = _Marshal(self.pairs)
        self._policy = policy  # keeps the device parameters alive
        self._o, self._t = _opts(node_limit, time_limit_s, tuning, policy, policy_depth,
                                 policy_mode, ordering, deadend_nodes, deadend_ratio)
        h = ctypes.c_void_p()
        st = self.lib.mcs_plan_create(len(self.pairs), self._m.G, self._m.H,
                                      ctypes.byref(self._o), ctypes.byref(h))
        if st < 0:
            raise McsError(st, _last_error())
        self.handle = h
        self.ws = None
        self.stream = None

    @property
    def workspace_bytes(self) -> int:
        return int(self.lib.mcs_plan_workspace_size(self.handle))

    def upload(self, stream=None):
        torch = _torch()
        nbytes = self.workspace_bytes
        self.ws = torch.empty(nbytes + 256, dtype=torch.uint8, device="cuda")
        base = self.ws.data_ptr()
        base = (base + 255) & ~255
        self.stream = stream if stream is not None else torch.cuda.current_stream()
        st = self.lib.mcs_plan_upload(self.handle, ctypes.c_void_p(base), nbytes,
                                      ctypes.c_void_p(self.stream.cuda_stream))
        if st < 0:
            raise McsError(st, _last_error())
        return self

    def run(self):
        st = self.lib.mcs_plan_run(self.handle, ctypes.c_void_p(self.stream.cuda_stream))
        if st < 0:
            raise McsError(st, _last_error())

    def set_goals(self, goals):
        """mcs_plan_set_goals: goal[i] > 0 asks the next runs only whether
        instance i has a common induced subgraph of at least goal[i]
        vertices; 0 is a plain search, < 0 skips the instance."""
        if len(goals) != len(self.pairs):
            raise ValueError("one goal per instance")
        g = (ctypes.c_int32 * len(goals))(*[int(x) for x in goals])
        st = self.lib.mcs_plan_set_goals(self.handle, g, ctypes.c_void_p(self.stream.cuda_stream))
        if st < 0:
            raise McsError(st, _last_error())

    def results(self):
        r = _Results(self._m.sizes)
        st = self.lib.mcs_plan_results(self.handle, r.res,
                                       ctypes.c_void_p(self.stream.cuda_stream))
        if st < 0:
            raise McsError(st, _last_error())
        self.status = st
        return r.results()

    def stats(self) -> Stats:
        s = _abi.mcs_stats()
        st = self.lib.mcs_plan_stats(self.handle, ctypes.byref(s))
        if st < 0:
            raise McsError(st, _last_error())
        return Stats(int(s.nodes), int(s.batches), int(s.children), int(s.lane_slots),
                     int(s.donations), int(s.pops), int(s.waves), int(s.blocks),
                     int(s.lds_per_wave), int(s.stopped), float(s.kernel_ms),
                     float(s.busy_wave_s), int(s.hbm_frames), int(s.stack_classes),
                     int(s.max_stack_used), float(s.sleep_wave_s), int(s.lds_bytes),
                     int(s.node_classes))

    def close(self):
        if getattr(self, "handle", None):
            self.lib.mcs_plan_destroy(self.handle)
            self.handle = None

    def __del__(self):
        try:
            self.close()
        except Exception:
            pass


def solve_batch(pairs, node_limit=0, time_limit_s=0.0, tuning=None, with_stats=False,
                policy=None, policy_depth=1, policy_mode=0, ordering="degree",
                deadend_nodes=0, deadend_ratio=0):
    """MCS of every pair in one launch.  Returns a list of Result (and Stats)."""
    p = Plan(pairs, node_limit, time_limit_s, tuning, policy, policy_depth, policy_mode,
             ordering, deadend_nodes, deadend_ratio).upload()
    p.run()
    res = p.results()
    st = p.stats() if with_stats else None
    p.close()
    return (res, st) if with_stats else res


def solve_batch_static(pairs, node_limit=0, time_limit_s=0.0, tuning=None, ordering="degree",
                       deadend_nodes=0, deadend_ratio=0):
    """MCS of every pair in one launch on the library's static device scratch
    (mcs_solve_batch_static): no device memory is allocated.  Returns a list
    of Result."""
    lib = _abi.load()
    torch = _torch()
    pairs = list(pairs)
    m = _Marshal(pairs)
    o, _t = _opts(node_limit, time_limit_s, tuning, ordering=ordering,
                  deadend_nodes=deadend_nodes, deadend_ratio=deadend_ratio)
    r = _Results(m.sizes)
    stream = torch.cuda.current_stream()
    st = lib.mcs_solve_batch_static(len(pairs), m.G, m.H, ctypes.byref(o),
                                    ctypes.c_void_p(stream.cuda_stream), r.res)
    if st < 0:
        raise McsError(st, _last_error())
    return r.results()


GOAL_STRATEGIES = {"top-down": 0, "bisect": 1, "dead-end+1": 2, "dead-end*2": 3}


def solve_goals(pairs, strategy="top-down", node_limit=0, time_limit_s=0.0, tuning=None,
                with_launches=False, ordering="degree", deadend_nodes=0, deadend_ratio=0):
    """Goal-directed search (mcs_solve_goals): strategy "top-down" asks for
    the root bound, then one less, ...; "bisect" takes a node-limited plain
    run's size as a lower bound and binary-searches the goal; "dead-end+1"
    and "dead-end*2" run the plain search with the dead-end forecast
    (deadend_nodes, deadend_ratio) and answer each forecast by raising the
    incumbent by 1, or by an increment that doubles at each forecast, then
    binary-search once a raised bound proves unreachable."""
    import torch
    lib = _abi.load()
    _torch()
    pairs = list(pairs)
    m = _Marshal(pairs)
    o, _t = _opts(node_limit, time_limit_s, tuning, ordering=ordering,
                  deadend_nodes=deadend_nodes, deadend_ratio=deadend_ratio)
    nbytes = int(lib.mcs_workspace_size(len(pairs), m.G, m.H, ctypes.byref(o)))
    if nbytes == 0:
        raise McsError(-1, _last_error())
    ws = torch.empty(nbytes + 256, dtype=torch.uint8, device="cuda")
    base = (ws.data_ptr() + 255) & ~255
    stream = torch.cuda.current_stream()
    r = _Results(m.sizes)
    launches = ctypes.c_int32(0)
    strat = GOAL_STRATEGIES[strategy]
    st = lib.mcs_solve_goals(len(pairs), m.G, m.H, ctypes.byref(o), strat, ctypes.c_void_p(base), nbytes,
                             ctypes.c_void_p(stream.cuda_stream), r.res, ctypes.byref(launches))
    if st < 0:
        raise McsError(st, _last_error())
    out = r.results()
    return (out, int(launches.value)) if with_launches else out


def solve(G, H, **kw):
    """MCS of one pair."""
    out = solve_batch([(G, H)], **kw)
    return out[0] if not kw.get("with_stats") else (out[0][0], out[1])


def workspace_size(pairs, node_limit=0, time_limit_s=0.0, tuning=None) -> int:
    lib = _abi.load()
    m = _Marshal(pairs)
    o, _t = _opts(node_limit, time_limit_s, tuning)
    return int(lib.mcs_workspace_size(len(pairs), m.G, m.H, ctypes.byref(o)))
