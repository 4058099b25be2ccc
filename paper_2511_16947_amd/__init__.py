"""Python binding of libfinemoe (ctypes; calls that pass tensors through csrc/call.cpp): argument marshalling only.

Every step of the MoE-layer hot path (gate top-K, token scheduling, permute,
grouped SwiGLU expert FFN, combine, backward) runs in the HIP kernels behind the
C ABI declared in include/finemoe.h.  PyTorch is used for device memory and the
current stream, nothing else.  There is no CPU fallback: if the library has not
been built (python -m paper_2511_16947_amd.build) importing a function and
calling it raises.
"""
from __future__ import annotations

import ctypes
import os
from dataclasses import dataclass
from functools import cached_property
from importlib.machinery import EXTENSION_SUFFIXES

import torch

_HERE = os.path.dirname(os.path.abspath(__file__))
LIB_PATH = os.path.join(_HERE, "libfinemoe.so")
CALL_PATH = os.path.join(_HERE, "_call" + EXTENSION_SUFFIXES[0])      # (built against this interpreter's headers, for it alone)

FINE_OK = 0
FINE_INVALID_ARG = -1
FINE_UNSUPPORTED = -2
FINE_WORKSPACE_TOO_SMALL = -3
FINE_INFEASIBLE = -4
FINE_HIP_ERROR = -5
FINE_F32, FINE_BF16 = 0, 1
FLAG_LOCALITY = 1
FLAG_ACT_SAVE_H = 16
# measurement and test switches (include/finemoe_measure.h; not part of the contract)
FLAG_SIMPLE_FFN, FLAG_ONLY_GEMM1, FLAG_ONLY_GEMM2 = 2, 4, 8
FLAG_TILE_SHIFT, FLAG_BWD_STAGE_SHIFT = 8, 12
WS_TOPK, WS_SCHED, WS_FFN, WS_BACKWARD = 0, 1, 2, 3

EXPORTS = ["fine_version", "fine_last_hip_error", "fine_workspace_bytes", "fine_topk", "fine_sched",
           "fine_sched_warm", "fine_sched_static", "fine_sched_comm", "fine_comm_replica_loads_host",
           "fine_permute", "fine_grouped_ffn", "fine_combine", "fine_backward", "fine_cayley_placement", "fine_replica_counts",
           "fine_eval_placements", "fine_place_search"]


class FineError(RuntimeError):
    def __init__(self, fn: str, code: int, hip: int = 0):
        names = {-1: "INVALID_ARG", -2: "UNSUPPORTED", -3: "WORKSPACE_TOO_SMALL", -4: "INFEASIBLE", -5: "HIP_ERROR"}
        super().__init__("%s failed: %s (%d)%s" % (fn, names.get(code, "?"), code,
                                                   ", hipError %d" % hip if code == FINE_HIP_ERROR else ""))
        self.code = code


class _Shape(ctypes.Structure):
    _fields_ = [(n, ctypes.c_int32) for n in ("T", "d", "f", "E", "K", "G", "dtype", "flags")]


_lib = None
_call = None      # _call.call
_entry = {}       # of the loaded library's functions below: address and kinds
# What the entry points that take device memory are passed between the shape and the stream: t a tensor or None (NULL), i an integer
_KINDS = {"fine_topk": "t" * 6 + "i", "fine_sched": "t" * 12 + "i", "fine_sched_warm": "t" * 13 + "i", "fine_sched_static": "t" * 11,
          "fine_sched_comm": "ttiii" + "t" * 10 + "i", "fine_permute": "ttt", "fine_grouped_ffn": "i" + "t" * 8 + "i",
          "fine_combine": "tttt", "fine_backward": "i" + "t" * 16 + "iti", "fine_cayley_placement": "iiiiit",
          "fine_replica_counts": "tit", "fine_eval_placements": "itttt", "fine_place_search": "ttiiitttt"}


def load_library() -> ctypes.CDLL:
    """Loads libfinemoe.so from the package directory; raises if it is not built."""
    global _lib, _call, _entry
    if _lib is not None:
        return _lib
    for path in (LIB_PATH, CALL_PATH):
        if not os.path.exists(path):
            raise FileNotFoundError(
                "%s is missing: build it with `python -m paper_2511_16947_amd.build` (there is no fallback path)" % path)
    from ._call import call
    lib = ctypes.CDLL(LIB_PATH)
    vp, sz, i32 = ctypes.c_void_p, ctypes.c_size_t, ctypes.c_int32
    sp = ctypes.POINTER(_Shape)
    lib.fine_version.restype = ctypes.c_int
    lib.fine_version.argtypes = []
    lib.fine_last_hip_error.restype = ctypes.c_int
    lib.fine_last_hip_error.argtypes = []
    lib.fine_workspace_bytes.restype = sz
    lib.fine_workspace_bytes.argtypes = [sp, ctypes.c_int]
    lib.fine_topk.restype = ctypes.c_int
    lib.fine_topk.argtypes = [sp, vp, vp, vp, vp, vp, vp, sz, vp]
    lib.fine_sched.restype = ctypes.c_int
    lib.fine_sched.argtypes = [sp] + [vp] * 11 + [vp, sz, vp]
    lib.fine_sched_warm.restype = ctypes.c_int
    lib.fine_sched_warm.argtypes = [sp] + [vp] * 12 + [vp, sz, vp]
    lib.fine_sched_static.restype = ctypes.c_int
    lib.fine_sched_static.argtypes = [sp] + [vp] * 11 + [vp]
    lib.fine_sched_comm.restype = ctypes.c_int
    lib.fine_sched_comm.argtypes = [sp, vp, vp, i32, i32, i32] + [vp] * 9 + [vp, sz, vp]
    lib.fine_comm_replica_loads_host.restype = ctypes.c_int
    lib.fine_comm_replica_loads_host.argtypes = [i32, i32, vp, vp, vp, i32, i32, vp, vp]
    lib.fine_permute.restype = ctypes.c_int
    lib.fine_permute.argtypes = [sp, vp, vp, vp, vp]
    lib.fine_grouped_ffn.restype = ctypes.c_int
    lib.fine_grouped_ffn.argtypes = [sp, i32, vp, vp, vp, vp, vp, vp, vp, vp, sz, vp]
    lib.fine_combine.restype = ctypes.c_int
    lib.fine_combine.argtypes = [sp, vp, vp, vp, vp, vp]
    lib.fine_backward.restype = ctypes.c_int
    lib.fine_backward.argtypes = [sp, i32] + [vp] * 16 + [ctypes.c_int, vp, sz, vp]
    lib.fine_cayley_placement.restype = ctypes.c_int
    lib.fine_cayley_placement.argtypes = [sp, i32, vp, i32, vp, i32, vp, vp]
    lib.fine_replica_counts.restype = ctypes.c_int
    lib.fine_replica_counts.argtypes = [sp, vp, i32, vp, vp]
    lib.fine_eval_placements.restype = ctypes.c_int
    lib.fine_eval_placements.argtypes = [sp, i32, vp, vp, vp, vp, vp]
    lib.fine_place_search.restype = ctypes.c_int
    lib.fine_place_search.argtypes = [sp, vp, vp, i32, i32, ctypes.c_uint32, vp, vp, vp, vp, vp]
    _call, _entry = call, {name: (ctypes.cast(getattr(lib, name), vp).value, kinds) for name, kinds in _KINDS.items()}
    _lib = lib
    return lib


@dataclass(frozen=True)
class Shape:
    T: int
    d: int
    f: int
    E: int
    K: int
    G: int
    dtype: int = FINE_BF16
    flags: int = FLAG_LOCALITY

    @property
    def P(self) -> int:
        return self.T * self.K

    @property
    def torch_dtype(self) -> torch.dtype:
        return torch.float32 if self.dtype == FINE_F32 else torch.bfloat16

    @cached_property
    def _ref(self):
        # what every call passes on: made by the first one, since a Shape never changes
        return ctypes.byref(self._struct)

    @cached_property
    def _struct(self) -> _Shape:
        return self.c()

    @cached_property
    def _at(self) -> int:
        return ctypes.addressof(self._struct)

    def c(self) -> _Shape:
        return _Shape(self.T, self.d, self.f, self.E, self.K, self.G, self.dtype, self.flags)

    def __getstate__(self):      # (a ctypes reference cannot be copied: copies make their own)
        return {k: v for k, v in self.__dict__.items() if k not in ("_ref", "_struct", "_at")}


# The handle that torch.cuda.current_stream() wraps, without the wrapper (2.9 us a call, this 0.3).  Small layers are bound by
# the host: one pass of a 256-token fp32 layer on four ranks, eight calls and twelve launches, kept it busy for 91 us, with
# this, plain integers for pointers and the shape converted once 63 us.  The wrapper also refuses a child forked after the GPU
# was initialised, and the functions are private to torch: there it is the wrapper.
def _stream():
    try:
        if not torch._C._cuda_isInBadFork():
            return torch._C._cuda_getCurrentRawStream(torch._C._cuda_getDevice())
    except AttributeError:
        pass
    return torch.cuda.current_stream().cuda_stream


def _run(fn: str, shape: Shape, *args):
    """A call of an entry point whose pointers are device memory: device-resident contiguous tensors, None for NULL."""
    if _lib is None:
        load_library()
    rc = _call(*_entry[fn], _stream, shape._at, *args)
    if rc != FINE_OK:
        _check(fn, rc)


def _check(fn: str, rc: int):
    if rc != FINE_OK:
        raise FineError(fn, rc, load_library().fine_last_hip_error())


def fine_version() -> int:
    return load_library().fine_version()


def fine_workspace_bytes(shape: Shape, which: int) -> int:
    return int(load_library().fine_workspace_bytes(shape._ref, which))


def alloc_workspace(shape: Shape, which: int, device="cuda") -> torch.Tensor:
    n = fine_workspace_bytes(shape, which)
    if n == 0:
        raise FineError("fine_workspace_bytes", FINE_INVALID_ARG)
    return torch.empty(n, dtype=torch.uint8, device=device)


def fine_topk(shape: Shape, x, w_router, bias, topk_idx, topk_w, ws=None):
    _run("fine_topk", shape, x, w_router, bias, topk_idx, topk_w, ws, 0 if ws is None else ws.numel())


def fine_sched(shape: Shape, topk_idx, place, load, input_eg, x_eg, max_load, pair_dst, row_of_pair, pair_of_row,
               seg_off, rank_off, ws):
    _run("fine_sched", shape, topk_idx, place, load, input_eg, x_eg, max_load, pair_dst, row_of_pair, pair_of_row,
         seg_off, rank_off, ws, ws.numel())


def fine_sched_warm(shape: Shape, topk_idx, place, x_prev, load, input_eg, x_eg, max_load, pair_dst, row_of_pair,
                    pair_of_row, seg_off, rank_off, ws):
    _run("fine_sched_warm", shape, topk_idx, place, x_prev, load, input_eg, x_eg, max_load, pair_dst, row_of_pair,
         pair_of_row, seg_off, rank_off, ws, ws.numel())


def fine_sched_static(shape: Shape, topk_idx, place, load, input_eg, x_eg, max_load, pair_dst, row_of_pair, pair_of_row,
                      seg_off, rank_off):
    _run("fine_sched_static", shape, topk_idx, place, load, input_eg, x_eg, max_load, pair_dst, row_of_pair,
         pair_of_row, seg_off, rank_off)


def fine_sched_comm(shape: Shape, topk_idx, place, alpha_num: int, alpha_den: int, ranks_per_node: int, load, input_eg,
                    x_eg, comp_comm, pair_dst, row_of_pair, pair_of_row, seg_off, rank_off, ws):
    _run("fine_sched_comm", shape, topk_idx, place, alpha_num, alpha_den, ranks_per_node, load, input_eg, x_eg,
         comp_comm, pair_dst, row_of_pair, pair_of_row, seg_off, rank_off, ws, ws.numel())


def fine_comm_replica_loads_host(load, input_eg, place, alpha_num: int, alpha_den: int):
    """Host arrays in (anything numpy converts), (x_eg[E,G] int32, (C*, M*)) out; marshalling only."""
    import numpy as np
    load = np.ascontiguousarray(load, dtype=np.int32)
    input_eg = np.ascontiguousarray(input_eg, dtype=np.int32)
    place = np.ascontiguousarray(place, dtype=np.uint8)
    E, G = place.shape
    x = np.zeros((E, G), dtype=np.int32)
    cc = np.zeros(2, dtype=np.int32)
    rc = load_library().fine_comm_replica_loads_host(E, G, load.ctypes.data, input_eg.ctypes.data, place.ctypes.data,
                                                     alpha_num, alpha_den, x.ctypes.data, cc.ctypes.data)
    _check("fine_comm_replica_loads_host", rc)
    return x, (int(cc[0]), int(cc[1]))


def fine_permute(shape: Shape, x, pair_of_row, x_perm):
    _run("fine_permute", shape, x, pair_of_row, x_perm)


def fine_grouped_ffn(shape: Shape, rank: int, x_perm, w_gate, w_up, w_down, seg_off, y_perm, act_save, ws):
    _run("fine_grouped_ffn", shape, rank, x_perm, w_gate, w_up, w_down, seg_off, y_perm, act_save, ws, ws.numel())


def fine_combine(shape: Shape, y_perm, row_of_pair, topk_w, out):
    _run("fine_combine", shape, y_perm, row_of_pair, topk_w, out)


def fine_backward(shape: Shape, rank: int, d_out, x_perm, y_perm, act_save, w_gate, w_up, w_down, row_of_pair,
                  pair_of_row, seg_off, topk_w, d_x, d_topk_w, d_w_gate, d_w_up, d_w_down, accumulate: bool, ws):
    _run("fine_backward", shape, rank, d_out, x_perm, y_perm, act_save, w_gate, w_up, w_down, row_of_pair,
         pair_of_row, seg_off, topk_w, d_x, d_topk_w, d_w_gate, d_w_up, d_w_down, 1 if accumulate else 0, ws,
         ws.numel())


def fine_cayley_placement(shape: Shape, orders, gens, complete: int, place):
    """orders: sequence of ints; gens: sequence of tuples of len(orders) ints (host data); place: device tensor."""
    k = len(orders)
    o = (ctypes.c_int32 * k)(*[int(v) for v in orders])
    flat = [int(v) for s in gens for v in s]
    assert len(flat) == k * len(gens)
    g = (ctypes.c_int32 * max(1, len(flat)))(*flat)
    _run("fine_cayley_placement", shape, k, ctypes.addressof(o), len(gens), ctypes.addressof(g), complete, place)


def fine_replica_counts(shape: Shape, load, slots: int, counts):
    _run("fine_replica_counts", shape, load, slots, counts)


def fine_eval_placements(shape: Shape, n: int, place, load, m_num, m_den):
    _run("fine_eval_placements", shape, n, place, load, m_num, m_den)


def fine_place_search(shape: Shape, load, counts, slots: int, n: int, seed: int, m_num, m_den, best, place):
    _run("fine_place_search", shape, load, counts, slots, n, seed & 0xFFFFFFFF, m_num, m_den, best, place)


# ---------------------------------------------------------------------------
# Buffer bundles (allocation only; no arithmetic)
# ---------------------------------------------------------------------------

class SchedBuffers:
    """Device tensors for the outputs of fine_sched plus its workspace."""

    def __init__(self, shape: Shape, device="cuda"):
        i32 = dict(dtype=torch.int32, device=device)
        E, G, P = shape.E, shape.G, shape.P
        self.load = torch.empty(E, **i32)
        self.input_eg = torch.empty(E, G, **i32)
        self.x_eg = torch.empty(E, G, **i32)
        self.max_load = torch.empty(1, **i32)
        self.pair_dst = torch.empty(P, **i32)
        self.row_of_pair = torch.empty(P, **i32)
        self.pair_of_row = torch.empty(P, **i32)
        self.seg_off = torch.empty(G, E + 1, **i32)
        self.rank_off = torch.empty(G + 1, **i32)
        self.ws = alloc_workspace(shape, WS_SCHED, device)

    def run(self, shape: Shape, topk_idx, place=None, warm: bool = False):
        """warm: start from the replica loads this object holds from its last run."""
        fine_sched_warm(shape, topk_idx, place, self.x_eg if warm else None, self.load, self.input_eg, self.x_eg, self.max_load, self.pair_dst,
                   self.row_of_pair, self.pair_of_row, self.seg_off, self.rank_off, self.ws)


def shape_of(cfg, flags: int = FLAG_LOCALITY) -> Shape:
    """Shape from a workload LayerConfig (duck typed: T, d, f, E, K, G, dtype)."""
    return Shape(cfg.T, cfg.d, cfg.f, cfg.E, cfg.K, cfg.G, FINE_F32 if cfg.dtype == "f32" else FINE_BF16, flags)
