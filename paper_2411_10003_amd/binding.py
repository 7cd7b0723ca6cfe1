"""Thin ctypes binding of libmoehot.so: the same entry points as include/moehot.h, taking torch
tensors.  Argument marshalling only -- every step of the layer runs in the HIP kernels of the
library.  PyTorch is used for device memory and streams.  There is no CPU or eager fallback: if
the library has not been built, `load()` raises.
"""
from __future__ import annotations

import ctypes
import importlib.util
import operator
import os
from typing import Dict, Optional

import torch

_HERE = os.path.dirname(os.path.abspath(__file__))
LIB_PATH = os.path.join(_HERE, "libmoehot.so")
PYCALL_PATH = os.path.join(_HERE, "_pycall.so")

MOE_F32, MOE_BF16 = 0, 1
MOE_ACT_GELU, MOE_ACT_SWIGLU = 0, 1
DTYPES = {"f32": MOE_F32, "bf16": MOE_BF16}
ACTS = {"gelu": MOE_ACT_GELU, "swiglu": MOE_ACT_SWIGLU}
TORCH_DTYPE = {MOE_F32: torch.float32, MOE_BF16: torch.bfloat16}

EXPORTS = [
    "moe_create", "moe_destroy", "moe_workspace_bytes", "moe_status_string", "moe_last_hip_error",
    "moe_read_status", "moe_gate_topk", "moe_expert_counts", "moe_dispatch", "moe_expert_ffn_fwd",
    "moe_combine", "moe_combine_bwd", "moe_expert_ffn_bwd", "moe_dispatch_bwd", "moe_gate_bwd",
    "moe_plan", "moe_gate_bwd_params", "moe_input_grad", "moe_expert_ffn_bwd_acc", "moe_trans", "moe_recv_layout",
    "moe_dispatch_after_counts", "moe_set_act_saved", "moe_expert_counts_static", "moe_agg", "moe_calib_copy", "moe_calib_mfma",
    "moe_calib_round_bf16",
]


class MoeError(RuntimeError):
    def __init__(self, status: int, where: str, detail: str = ""):
        self.status = status
        super().__init__(f"{where}: status {status} ({detail})")


class _Shape(ctypes.Structure):
    _fields_ = [(n, ctypes.c_int) for n in ("T", "d", "h", "E", "k", "P", "self", "G", "dtype", "act", "renorm")]


class _Layout(ctypes.Structure):
    _fields_ = [(n, ctypes.c_void_p) for n in
                ("slot_of_expert", "slot_offsets", "dest_offsets", "dest_slots", "pos", "perm")]


class _Planner(ctypes.Structure):
    _fields_ = [(n, ctypes.c_int) for n in ("D", "E", "n", "overlap")] + \
               [(n, ctypes.c_double) for n in ("alpha", "size_input", "size_params", "size_grads", "B", "t", "T_FNEC", "T_BNEC")]


class _PlanOut(ctypes.Structure):
    _fields_ = [(n, ctypes.c_void_p) for n in ("expert_dest", "selected", "skipped", "H", "R", "times", "info")]


_raw_stream, _current_device = getattr(torch._C, "_cuda_getCurrentRawStream", None), getattr(torch._C, "_cuda_getDevice", None)
_lib = _call_class = None


def load() -> ctypes.CDLL:
    """Load the HIP library.  Raises if it is missing: nothing else can compute the layer."""
    global _lib
    if _lib is None:
        if not os.path.exists(LIB_PATH):
            raise ImportError(f"{LIB_PATH} is not built; run `python -m paper_2411_10003_amd.build`")
        lib = ctypes.CDLL(LIB_PATH)
        vp, ip = ctypes.c_void_p, ctypes.c_int
        lib.moe_create.argtypes = [ctypes.POINTER(vp), ctypes.POINTER(_Shape)]
        lib.moe_destroy.argtypes = [vp]
        lib.moe_workspace_bytes.argtypes = [vp, ctypes.POINTER(ctypes.c_size_t)]
        lib.moe_status_string.argtypes = [ip]
        lib.moe_status_string.restype = ctypes.c_char_p
        lib.moe_read_status.argtypes = [vp, vp, vp, ctypes.POINTER(ip)]
        lib.moe_gate_topk.argtypes = [vp] * 8
        lib.moe_expert_counts.argtypes = [vp] * 5
        lib.moe_dispatch.argtypes = [vp, vp, vp, vp, vp, ctypes.POINTER(_Layout), vp, vp, vp]
        lib.moe_dispatch_after_counts.argtypes = [vp, vp, vp, vp, vp, ctypes.POINTER(_Layout), vp, vp, vp]
        lib.moe_set_act_saved.argtypes = [vp, ip]
        lib.moe_expert_counts_static.argtypes = [vp] * 4
        lib.moe_expert_ffn_fwd.argtypes = [vp, vp, ctypes.POINTER(_Layout)] + [vp] * 8
        lib.moe_combine.argtypes = [vp] * 6
        lib.moe_combine_bwd.argtypes = [vp] * 8
        lib.moe_expert_ffn_bwd.argtypes = [vp] * 5 + [ctypes.POINTER(_Layout)] + [vp] * 9
        lib.moe_expert_ffn_bwd_acc.argtypes = [vp] * 5 + [ctypes.POINTER(_Layout)] + [vp] * 9
        lib.moe_dispatch_bwd.argtypes = [vp] * 5
        lib.moe_gate_bwd.argtypes = [vp] * 6
        lib.moe_gate_bwd_params.argtypes = [vp] * 7
        lib.moe_input_grad.argtypes = [vp] * 7
        lib.moe_trans.argtypes = [vp, vp, vp, vp, vp, ip, ctypes.POINTER(vp), ctypes.POINTER(vp), ctypes.POINTER(ctypes.c_size_t), vp]
        lib.moe_agg.argtypes = [vp, vp, ip, ctypes.POINTER(vp), ctypes.POINTER(vp), ctypes.POINTER(ctypes.c_size_t), vp]
        lib.moe_calib_copy.argtypes = [vp, vp, ctypes.c_size_t, vp]
        lib.moe_calib_mfma.argtypes = [vp, ctypes.c_size_t, ip, ctypes.POINTER(ip), ctypes.POINTER(ip), vp]
        lib.moe_calib_round_bf16.argtypes = [vp, vp, ctypes.c_size_t, vp]
        lib.moe_recv_layout.argtypes = [vp, ctypes.POINTER(_Layout), vp, ctypes.POINTER(_Layout), vp]
        lib.moe_plan.argtypes = [ctypes.POINTER(_Planner), vp, ctypes.POINTER(_PlanOut), vp]
        _lib = lib
    return _lib


class PythonCall:
    """What the module of the native calls has as Call, where it is not built: the same arguments, checks and errors, in Python."""

    def __init__(self, entry: int, args: tuple, check):
        self._f, self._args, self._check = ctypes.CFUNCTYPE(ctypes.c_int, *[ctypes.c_void_p] * len(args))(entry), args, check
        self._n = sum(not isinstance(a, int) for a in args)

    def __call__(self, *given) -> int:
        if len(given) != self._n:
            raise TypeError(f"{self._n} positional arguments expected")
        it = iter(given)
        return self._f(*(a if isinstance(a, int) else self._pointer(next(it), a) for a in self._args))

    def _pointer(self, given, arg):
        if arg == "int":
            return operator.index(given)
        return None if given is None else self._check(given, *arg)


def _call_type():
    """The type of the calls: native, or in Python where the native ones are not built or were built for another torch."""
    global _call_class
    if _call_class is None:
        try:
            spec = importlib.util.spec_from_file_location("_pycall", PYCALL_PATH)
            module = importlib.util.module_from_spec(spec)
            spec.loader.exec_module(module)
            _call_class = module.Call
        except ImportError:
            _call_class = PythonCall
    return _call_class


def _ptr(t: Optional[torch.Tensor], dtype: torch.dtype, numel: int, name: str) -> Optional[int]:
    if t is None:
        return None
    if not t.is_cuda or not t.is_contiguous():
        raise ValueError(f"{name}: need a contiguous device tensor")
    if t.dtype != dtype:
        raise ValueError(f"{name}: dtype {t.dtype}, expected {dtype}")
    if t.numel() < numel:
        raise ValueError(f"{name}: {t.numel()} elements, need {numel}")
    return t.data_ptr()


def _stream() -> int:
    # The raw handle of the current stream.  torch.cuda.current_stream() builds a Stream object around it first: 2.9 us, a
    # third of the host time of a call; this takes 0.2 (the five calls of the tiny forward layer 43 -> 30 us).
    if _raw_stream is None or _current_device is None:
        return torch.cuda.current_stream().cuda_stream
    return _raw_stream(_current_device())


class PlanBuffers:
    """Device arrays moe_plan writes (see moe_plan_out_t)."""

    def __init__(self, D: int, E: int, device="cuda:0"):
        self.D, self.E = D, E
        self.expert_dest = torch.zeros(D, E, dtype=torch.int32, device=device)
        self.selected = torch.zeros(E, dtype=torch.int32, device=device)
        self.skipped = torch.zeros(E, dtype=torch.int64, device=device)      # bit masks, read as unsigned
        self.H = torch.zeros(D, dtype=torch.int64, device=device)
        self.R = torch.zeros(D, dtype=torch.int64, device=device)
        self.times = torch.zeros(2 + E, dtype=torch.float64, device=device)
        self.info = torch.zeros(2, dtype=torch.int32, device=device)
        self.c = _PlanOut(*(t.data_ptr() for t in (self.expert_dest, self.selected, self.skipped, self.H, self.R,
                                                   self.times, self.info)))


def plan(gating: torch.Tensor, out: PlanBuffers, *, n: int, overlap: bool, alpha: float, size_input: float,
         size_params: float, size_grads: float, B: float, t: float, T_FNEC: float = 0.0, T_BNEC: float = 0.0) -> None:
    """moe_plan: greedy search for a lightweight expert placement on the device (argument marshalling only)."""
    lib = load()
    D, E = out.D, out.E
    g = _ptr(gating, torch.int32, D * E, "gating")
    cfg = _Planner(D, E, int(n), int(bool(overlap)), float(alpha), float(size_input), float(size_params),
                   float(size_grads), float(B), float(t), float(T_FNEC), float(T_BNEC))
    rc = lib.moe_plan(ctypes.byref(cfg), g, ctypes.byref(out.c), _stream())
    if rc != 0:
        raise MoeError(rc, "moe_plan", lib.moe_status_string(rc).decode())


def calib_copy(src: torch.Tensor, dst: torch.Tensor) -> None:
    """moe_calib_copy: a plain streaming copy of src into dst (uint8 tensors of the same size)."""
    lib = load()
    n = src.numel() * src.element_size()
    rc = lib.moe_calib_copy(_ptr(src, src.dtype, src.numel(), "src"), _ptr(dst, src.dtype, src.numel(), "dst"), n, _stream())
    if rc != 0:
        raise MoeError(rc, "moe_calib_copy", lib.moe_status_string(rc).decode())


def calib_mfma(out: torch.Tensor, iters: int) -> float:
    """moe_calib_mfma: enqueue the register-only bf16 MFMA loop; returns the flops it performs."""
    lib = load()
    blocks, threads = ctypes.c_int(0), ctypes.c_int(0)
    rc = lib.moe_calib_mfma(_ptr(out, torch.float32, 1, "out"), out.numel(), int(iters), ctypes.byref(blocks),
                            ctypes.byref(threads), _stream())
    if rc != 0:
        raise MoeError(rc, "moe_calib_mfma", lib.moe_status_string(rc).decode())
    return float(blocks.value) * (threads.value // 64) * iters * 16 * 16384.0


def calib_round_bf16(x: torch.Tensor, out: torch.Tensor) -> None:
    """moe_calib_round_bf16: out[i] (int16 bit patterns) = the library's fp32 -> bf16 rounding of x[i]."""
    lib = load()
    rc = lib.moe_calib_round_bf16(_ptr(x, torch.float32, 1, "x"), _ptr(out, torch.int16, x.numel(), "out"), x.numel(), _stream())
    if rc != 0:
        raise MoeError(rc, "moe_calib_round_bf16", lib.moe_status_string(rc).decode())


class Layout:
    """Device arrays of the send layout (see moe_layout_t)."""

    def __init__(self, E: int, P: int, A: int, device):
        i32 = dict(dtype=torch.int32, device=device)
        self.slot_of_expert = torch.zeros(E, **i32)
        self.slot_offsets = torch.zeros(E + 1, **i32)
        self.dest_offsets = torch.zeros(P + 1, **i32)
        self.dest_slots = torch.zeros(P + 1, **i32)
        self.pos = torch.zeros(A, **i32)
        self.perm = torch.zeros(A, **i32)
        self.c = _Layout(*(t.data_ptr() for t in (self.slot_of_expert, self.slot_offsets, self.dest_offsets,
                                                  self.dest_slots, self.pos, self.perm)))


# What stands at the arguments of each entry point between the handle and the stream: tensors by dtype, least number of elements and
# name; "int" an address that is given at the call.  (e: the handle's element type, f and i: fp32 and int32, m: all weights of a kind.)
# One call object per handle and entry point.
def _dispatch_spec(s, e, f, i, m):
    return (i, s.E, "expert_dest"), (e, s.T * s.d, "X"), (i, s.A, "idx"), (i, s.E, "counts"), "int", (e, s.A * s.d, "Xp"), "int"


def _bwd_spec(s, e, f, i, m):
    rows, hidden = s.A * s.d, s.A * s.h
    return ((e, rows, "dYp"), (e, rows, "Xp"), (e, hidden, "Z"), (e, hidden, "U"), "int", (e, m, "W1"), (e, m, "W2"), (e, m, "W3"), (e, rows, "dXp"),
            (f, m, "dW1"), (f, m, "dW2"), (f, m, "dW3"), "int")


_SPECS = {
    "moe_gate_topk": lambda s, e, f, i, m: ((e, s.T * s.d, "X"), (f, s.d * s.E, "Wg"), (f, s.E, "bg"), (f, s.T * s.E, "logits"), (i, s.A, "idx"), (f, s.A, "w")),
    "moe_expert_counts": lambda s, e, f, i, m: ((i, s.A, "idx"), (i, s.E, "counts"), "int"),
    "moe_dispatch": _dispatch_spec,
    "moe_dispatch_after_counts": _dispatch_spec,
    "moe_expert_ffn_fwd": lambda s, e, f, i, m: ((e, s.A * s.d, "Xp"), "int", (e, m, "W1"), (e, m, "W2"), (e, m, "W3"), (e, s.A * s.d, "Yp"),
                                                 (e, s.A * s.h, "Z"), (e, s.A * s.h, "U"), "int"),
    "moe_combine": lambda s, e, f, i, m: ((e, s.A * s.d, "Yp"), (i, s.A, "pos"), (f, s.A, "w"), (e, s.T * s.d, "out")),
    "moe_combine_bwd": lambda s, e, f, i, m: ((e, s.T * s.d, "dOut"), (e, s.A * s.d, "Yp"), (i, s.A, "pos"), (f, s.A, "w"), (e, s.A * s.d, "dYp"),
                                              (f, s.A, "dw")),
    "moe_expert_ffn_bwd": _bwd_spec,
    "moe_expert_ffn_bwd_acc": _bwd_spec,
    "moe_dispatch_bwd": lambda s, e, f, i, m: ((e, s.A * s.d, "dXp"), (i, s.A, "pos"), (e, s.T * s.d, "dX")),
    "moe_gate_bwd": lambda s, e, f, i, m: ((f, s.A, "dw"), (f, s.T * s.E, "logits"), (i, s.A, "idx"), (f, s.T * s.E, "dlogits")),
    "moe_gate_bwd_params": lambda s, e, f, i, m: ((e, s.T * s.d, "X"), (f, s.T * s.E, "dlogits"), (f, s.d * s.E, "dWg"), (f, s.E, "dbg"), "int"),
    "moe_input_grad": lambda s, e, f, i, m: ((e, s.A * s.d, "dXp"), (i, s.A, "pos"), (f, s.T * s.E, "dlogits"), (f, s.d * s.E, "Wg"), (e, s.T * s.d, "dX")),
}
_entries: Dict[str, int] = {}


def _entry(name: str) -> int:
    """The address of an entry point."""
    if name not in _entries:
        _entries[name] = ctypes.cast(getattr(load(), name), ctypes.c_void_p).value
    return _entries[name]


class Handle:
    """A moe_handle_t plus its workspace.  Methods carry the names of the C entry points."""

    def __init__(self, *, T: int, d: int, h: int, E: int, k: int, P: int, self_dest: int, G: int,
                 dtype: str, act: str, renorm: int, device="cuda:0", alloc_workspace: bool = True):
        self.lib = load()
        self.shape = _Shape(T, d, h, E, k, P, self_dest, G, DTYPES[dtype], ACTS[act], renorm)
        self.T, self.d, self.h, self.E, self.k, self.P, self.G = T, d, h, E, k, P, G
        self.A = T * k
        self.swiglu = act == "swiglu"
        self.elt = TORCH_DTYPE[DTYPES[dtype]]
        self.device = torch.device(device)
        self._h = ctypes.c_void_p()
        self._check(self.lib.moe_create(ctypes.byref(self._h), ctypes.byref(self.shape)), "moe_create")
        n = ctypes.c_size_t()
        self._check(self.lib.moe_workspace_bytes(self._h, ctypes.byref(n)), "moe_workspace_bytes")
        self.workspace_bytes = n.value
        self.ws = torch.empty(n.value, dtype=torch.uint8, device=self.device) if alloc_workspace else None
        self._calls: Dict[str, object] = {}

    def close(self):
        if self._h:
            self._calls = {}                               # they hold its address
            self.lib.moe_destroy(self._h)
            self._h = ctypes.c_void_p()

    def __del__(self):
        try:
            self.close()
        except Exception:
            pass

    def _check(self, rc: int, where: str):
        if rc != 0:
            detail = self.lib.moe_status_string(rc).decode()
            if rc == -7:
                detail += f", hipError {self.lib.moe_last_hip_error()}"
            raise MoeError(rc, where, detail)

    def _ws(self) -> int:
        if self.ws is None:
            raise ValueError("no workspace attached")
        return self.ws.data_ptr()

    def new_layout(self) -> Layout:
        return Layout(self.E, self.P, self.A, self.device)

    # ---- the entry points ---------------------------------------------------------------
    def read_status(self) -> int:
        v = ctypes.c_int(0)
        self._check(self.lib.moe_read_status(self._h, self._ws(), _stream(), ctypes.byref(v)), "moe_read_status")
        return v.value

    def _spec(self, name: str):
        return _SPECS[name](self, self.elt, torch.float32, torch.int32, self.G * self.d * self.h)

    def _call(self, name: str, *args):
        call = self._calls.get(name)
        if call is None:
            call = self._calls[name] = _call_type()(_entry(name), (self._h.value or 0, *self._spec(name), "int"), _ptr)
        rc = call(*args, _stream())
        if rc != 0:
            self._check(rc, name)

    def gate_topk(self, X, Wg, bg, logits, idx, w):
        self._call("moe_gate_topk", X, Wg, bg, logits, idx, w)

    def expert_counts(self, idx, counts):
        self._call("moe_expert_counts", idx, counts, self._ws())

    def expert_counts_static(self, idx, counts):
        i32 = torch.int32
        self._check(self.lib.moe_expert_counts_static(self._h, _ptr(idx, i32, self.A, "idx"), _ptr(counts, i32, self.E, "counts"),
                                                      _stream()), "moe_expert_counts_static")

    def dispatch(self, expert_dest, X, idx, counts, layout: Layout, Xp, after_counts: bool = False):
        self._call("moe_dispatch_after_counts" if after_counts else "moe_dispatch", expert_dest, X, idx, counts,
                   ctypes.addressof(layout.c), Xp, self._ws())

    def dispatch_after_counts(self, expert_dest, X, idx, counts, layout: Layout, Xp):
        self.dispatch(expert_dest, X, idx, counts, layout, Xp, after_counts=True)

    def set_act_saved(self, saved: bool):
        self._check(self.lib.moe_set_act_saved(self._h, int(bool(saved))), "moe_set_act_saved")

    def expert_ffn_fwd(self, Xp, layout: Layout, W1, W2, W3, Yp, Z, U):
        self._call("moe_expert_ffn_fwd", Xp, ctypes.addressof(layout.c), W1, W2, W3, Yp, Z, U, self._ws())

    def combine(self, Yp, pos, w, out):
        self._call("moe_combine", Yp, pos, w, out)

    def combine_bwd(self, dOut, Yp, pos, w, dYp, dw):
        self._call("moe_combine_bwd", dOut, Yp, pos, w, dYp, dw)

    def expert_ffn_bwd(self, dYp, Xp, Z, U, layout: Layout, W1, W2, W3, dXp, dW1, dW2, dW3, accumulate: bool = False):
        self._call("moe_expert_ffn_bwd_acc" if accumulate else "moe_expert_ffn_bwd", dYp, Xp, Z, U, ctypes.addressof(layout.c),
                   W1, W2, W3, dXp, dW1, dW2, dW3, self._ws())

    def expert_ffn_bwd_acc(self, *args):
        self.expert_ffn_bwd(*args, accumulate=True)

    def dispatch_bwd(self, dXp, pos, dX):
        self._call("moe_dispatch_bwd", dXp, pos, dX)

    def gate_bwd(self, dw, logits, idx, dlogits):
        self._call("moe_gate_bwd", dw, logits, idx, dlogits)

    def trans(self, expert_dest, slot_expert, pools, groups, pool_version=None, slot_version=None):
        """moe_trans: gather the hosted experts' tensors from the pools into the group slots."""
        n = len(pools)
        per = [p.numel() // self.E * p.element_size() for p in pools]
        for p, g, b in zip(pools, groups, per):
            if not (p.is_cuda and g.is_cuda and p.is_contiguous() and g.is_contiguous()):
                raise ValueError("trans: need contiguous device tensors")
            if p.numel() % self.E or g.numel() * g.element_size() < self.G * b or p.dtype != g.dtype:
                raise ValueError("trans: pool / group sizes do not match")
        pa = (ctypes.c_void_p * n)(*(p.data_ptr() for p in pools))
        ga = (ctypes.c_void_p * n)(*(g.data_ptr() for g in groups))
        ba = (ctypes.c_size_t * n)(*per)
        self._check(self.lib.moe_trans(
            self._h, _ptr(expert_dest, torch.int32, self.E, "expert_dest"), _ptr(pool_version, torch.int32, self.E, "pool_version"),
            _ptr(slot_expert, torch.int32, self.G, "slot_expert"), _ptr(slot_version, torch.int32, self.G, "slot_version"),
            n, pa, ga, ba, _stream()), "moe_trans")

    def agg(self, expert_dest, group_grads, pool_grads):
        """moe_agg: add the hosted groups' weight gradients to the per-expert gradient pools."""
        n = len(group_grads)
        per = [p.numel() // self.E for p in pool_grads]
        for p, g, b in zip(pool_grads, group_grads, per):
            if not (p.is_cuda and g.is_cuda and p.is_contiguous() and g.is_contiguous()):
                raise ValueError("agg: need contiguous device tensors")
            if p.dtype != torch.float32 or g.dtype != torch.float32 or p.numel() % self.E or g.numel() < self.G * b:
                raise ValueError("agg: pool / group sizes or dtypes do not match")
        ga = (ctypes.c_void_p * n)(*(g.data_ptr() for g in group_grads))
        pa = (ctypes.c_void_p * n)(*(p.data_ptr() for p in pool_grads))
        ba = (ctypes.c_size_t * n)(*per)
        self._check(self.lib.moe_agg(self._h, _ptr(expert_dest, torch.int32, self.E, "expert_dest"), n, ga, pa, ba, _stream()),
                    "moe_agg")

    def recv_layout(self, local: Layout, recv_offsets, out: Layout):
        self._check(self.lib.moe_recv_layout(
            self._h, ctypes.byref(local.c), _ptr(recv_offsets, torch.int32, self.G + 1, "recv_offsets"),
            ctypes.byref(out.c), _stream()), "moe_recv_layout")

    def gate_bwd_params(self, X, dlogits, dWg, dbg):
        self._call("moe_gate_bwd_params", X, dlogits, dWg, dbg, self._ws())

    def input_grad(self, dXp, pos, dlogits, Wg, dX):
        self._call("moe_input_grad", dXp, pos, dlogits, Wg, dX)


class LayerBuffers:
    """Every device buffer of one layer pass, allocated once (nothing is allocated per step)."""

    def __init__(self, hd: Handle, backward: bool):
        dev, e = hd.device, hd.elt
        f32 = dict(dtype=torch.float32, device=dev)
        i32 = dict(dtype=torch.int32, device=dev)
        T, d, h, E, A, G = hd.T, hd.d, hd.h, hd.E, hd.A, hd.G
        self.logits = torch.empty(T, E, **f32)
        self.idx = torch.empty(T, hd.k, **i32)
        self.w = torch.empty(T, hd.k, **f32)
        self.counts = torch.empty(E, **i32)
        self.layout = hd.new_layout()
        self.Xp = torch.empty(A, d, dtype=e, device=dev)
        self.Yp = torch.empty(A, d, dtype=e, device=dev)
        self.Z = torch.empty(A, h, dtype=e, device=dev)
        self.U = torch.empty(A, h, dtype=e, device=dev) if hd.swiglu else None
        self.out = torch.empty(T, d, dtype=e, device=dev)
        if backward:
            self.dYp = torch.empty(A, d, dtype=e, device=dev)
            self.dw = torch.empty(T, hd.k, **f32)
            self.dXp = torch.empty(A, d, dtype=e, device=dev)
            self.dW1 = torch.empty(G, d, h, **f32)
            self.dW2 = torch.empty(G, h, d, **f32)
            self.dW3 = torch.empty(G, d, h, **f32) if hd.swiglu else None
            self.dX = torch.empty(T, d, dtype=e, device=dev)
            self.dlogits = torch.empty(T, E, **f32)


def layer_forward(hd: Handle, b: LayerBuffers, X, Wg, bg, expert_dest, W1, W2, W3):
    """The forward calls in order; rows of other destinations in b.Yp are left as the caller set them."""
    hd.gate_topk(X, Wg, bg, b.logits, b.idx, b.w)
    hd.expert_counts(b.idx, b.counts)
    hd.dispatch_after_counts(expert_dest, X, b.idx, b.counts, b.layout, b.Xp)   # same idx, same workspace, nothing in between
    hd.expert_ffn_fwd(b.Xp, b.layout, W1, W2, W3, b.Yp, b.Z, b.U)
    hd.combine(b.Yp, b.layout.pos, b.w, b.out)


def layer_backward(hd: Handle, b: LayerBuffers, dOut, W1, W2, W3):
    """The backward calls in order; rows of other destinations in b.dXp are left as the caller set them."""
    hd.combine_bwd(dOut, b.Yp, b.layout.pos, b.w, b.dYp, b.dw)
    hd.expert_ffn_bwd(b.dYp, b.Xp, b.Z, b.U, b.layout, W1, W2, W3, b.dXp, b.dW1, b.dW2, b.dW3)
    hd.dispatch_bwd(b.dXp, b.layout.pos, b.dX)
    hd.gate_bwd(b.dw, b.logits, b.idx, b.dlogits)
