"""ctypes binding of libgrpic.so (C ABI in include/grpic.h).

Argument marshalling only: every function here checks tensor devices, dtypes
and sizes, builds the C structures and calls the function of the same name in
the library, which does all the work on the GPU.  There is no fallback: if
the library is missing, ``lib()`` raises.
"""
from __future__ import annotations

import ctypes
import os

import numpy as np
import torch

PKG = os.path.dirname(os.path.abspath(__file__))
LIB_PATH = os.path.join(PKG, "libgrpic.so")

GRPIC_OK, GRPIC_EINVAL, GRPIC_ERANGE, GRPIC_ENOMEM, GRPIC_EHIP = 0, -1, -2, -3, -4
GRPIC_FP64, GRPIC_FP32_SPLIT = 0, 1
GRPIC_MAX_SPECIES = 8
GRPIC_NCOUNTERS = 5
COUNTER_NAMES = ("out", "bad", "reflected", "live_steps", "spilled")
GRPIC_NQCOUNTERS = 3
QCOUNTER_NAMES = ("emitted", "converted", "dropped")

PARTICLE_KEYS = ("cell", "xr", "xth", "ur", "uth", "uph", "w", "sp")
REAL_KEYS = ("xr", "xth", "ur", "uth", "uph", "w")


class grpic_metric(ctypes.Structure):
    _fields_ = [("a", ctypes.c_double), ("M", ctypes.c_double)]


class grpic_grid(ctypes.Structure):
    _fields_ = [("nr", ctypes.c_int32), ("nth", ctypes.c_int32), ("guard", ctypes.c_int32),
                ("pitch", ctypes.c_int32), ("lnr0", ctypes.c_double), ("dlnr", ctypes.c_double),
                ("dth", ctypes.c_double)]


class grpic_species(ctypes.Structure):
    _fields_ = [("q", ctypes.c_double), ("m", ctypes.c_double), ("massless", ctypes.c_int32),
                ("reserved", ctypes.c_int32)]


class grpic_particles(ctypes.Structure):
    _fields_ = [("n", ctypes.c_int64), ("cell", ctypes.c_void_p), ("xr", ctypes.c_void_p),
                ("xth", ctypes.c_void_p), ("ur", ctypes.c_void_p), ("uth", ctypes.c_void_p),
                ("uph", ctypes.c_void_p), ("w", ctypes.c_void_p), ("sp", ctypes.c_void_p),
                ("phi", ctypes.c_void_p), ("precision", ctypes.c_int32), ("reserved", ctypes.c_int32),
                ("tag", ctypes.c_void_p)]


class grpic_qed(ctypes.Structure):
    _fields_ = [("gamma_thr", ctypes.c_double), ("eps_ph", ctypes.c_double), ("tau", ctypes.c_double),
                ("seed", ctypes.c_uint64), ("electron_sp", ctypes.c_int32), ("positron_sp", ctypes.c_int32),
                ("photon_sp", ctypes.c_int32), ("reserved", ctypes.c_int32)]


class grpic_fields(ctypes.Structure):
    _fields_ = [("D", ctypes.c_void_p * 3), ("B", ctypes.c_void_p * 3)]


class grpic_current(ctypes.Structure):
    _fields_ = [("Fr", ctypes.c_void_p), ("Fth", ctypes.c_void_p), ("Gph", ctypes.c_void_p)]


class grpic_momentum_grads(ctypes.Structure):
    _fields_ = [("ur", ctypes.c_void_p), ("uth", ctypes.c_void_p), ("uph", ctypes.c_void_p)]


class grpic_field_grads(ctypes.Structure):
    _fields_ = [("D", ctypes.c_void_p * 3), ("B", ctypes.c_void_p * 3)]


class grpic_backward_range(ctypes.Structure):
    _fields_ = [("first", ctypes.c_int64), ("count", ctypes.c_int64), ("field_step_stride", ctypes.c_size_t),
                ("grad_step_stride", ctypes.c_size_t)]


class grpic_field_state(ctypes.Structure):
    _fields_ = [("D", ctypes.c_void_p * 3), ("B", ctypes.c_void_p * 3)]


EXPORTED = ("grpic_push_deposit", "grpic_push_deposit_vay", "grpic_push_deposit_spline3", "grpic_charge3",
            "grpic_push_deposit_qed", "grpic_qed_workspace_bytes", "grpic_sort_noalloc", "grpic_push_deposit_backward_range",
            "grpic_push_deposit_backward", "grpic_checkpoint_bytes",
            "grpic_backward_workspace_bytes", "grpic_charge", "grpic_sort", "grpic_sort_workspace_bytes",
            "grpic_tiling_bytes", "grpic_crossing_time", "grpic_last_error", "grpic_version",
            "grpic_field_tables_bytes", "grpic_field_workspace_bytes", "grpic_field_tables", "grpic_field_step")


class GrpicError(RuntimeError):
    def __init__(self, code: int, msg: str):
        super().__init__(f"grpic error {code}: {msg}")
        self.code = code


_lib = None


def lib():
    """The loaded libgrpic.so; raises if it has not been built."""
    global _lib
    if _lib is None:
        if not os.path.exists(LIB_PATH):
            raise RuntimeError(f"{LIB_PATH} is not built: run `python -m paper_2503_04558_amd.build`")
        L = ctypes.CDLL(LIB_PATH)
        vp, i32, i64, f64 = ctypes.c_void_p, ctypes.c_int, ctypes.c_int64, ctypes.c_double
        sz = ctypes.c_size_t
        L.grpic_push_deposit.argtypes = [vp, vp, vp, i32, vp, vp, vp, vp, f64, i32, i32, vp, sz, i32, vp, vp]
        L.grpic_push_deposit_backward.argtypes = [vp, vp, vp, i32, vp, vp, vp, f64, i32, i32, vp, sz, i32, vp, sz,
                                                  vp, vp, vp]
        L.grpic_push_deposit_backward.restype = ctypes.c_int
        L.grpic_push_deposit_backward_range.argtypes = [vp, vp, vp, i32, vp, vp, vp, f64, i32, i32, vp, sz, i32, vp,
                                                        vp, sz, vp, vp, vp]
        L.grpic_push_deposit_backward_range.restype = ctypes.c_int
        L.grpic_checkpoint_bytes.argtypes = [i64, i32, i32]
        L.grpic_checkpoint_bytes.restype = sz
        L.grpic_backward_workspace_bytes.argtypes = [vp, i64, i32]
        L.grpic_backward_workspace_bytes.restype = sz
        L.grpic_push_deposit.restype = ctypes.c_int
        L.grpic_push_deposit_vay.argtypes = [vp, vp, vp, i32, vp, vp, vp, vp, f64, i32, i32, vp, vp]
        L.grpic_push_deposit_vay.restype = ctypes.c_int
        L.grpic_push_deposit_spline3.argtypes = [vp, vp, vp, i32, vp, vp, vp, vp, f64, i32, i32, vp, vp]
        L.grpic_push_deposit_spline3.restype = ctypes.c_int
        L.grpic_push_deposit_qed.argtypes = [vp, vp, vp, i32, vp, vp, vp, vp, f64, i64, i32, vp, vp, vp, sz, vp, vp,
                                             vp]
        L.grpic_push_deposit_qed.restype = ctypes.c_int
        L.grpic_qed_workspace_bytes.argtypes = [vp, i64]
        L.grpic_qed_workspace_bytes.restype = sz
        L.grpic_charge3.argtypes = [vp, vp, i32, vp, vp, vp]
        L.grpic_charge3.restype = ctypes.c_int
        L.grpic_charge.argtypes = [vp, vp, i32, vp, vp, vp]
        L.grpic_charge.restype = ctypes.c_int
        L.grpic_sort_workspace_bytes.argtypes = [vp, i64]
        L.grpic_sort_workspace_bytes.restype = ctypes.c_size_t
        L.grpic_sort.argtypes = [vp, vp, vp, vp, vp, ctypes.c_size_t, vp, ctypes.c_size_t, vp, vp]
        L.grpic_sort_noalloc.argtypes = [vp, vp, vp, vp, vp, ctypes.c_size_t, vp, vp]
        L.grpic_sort_noalloc.restype = ctypes.c_int
        L.grpic_tiling_bytes.argtypes = [vp, i64]
        L.grpic_tiling_bytes.restype = ctypes.c_size_t
        L.grpic_sort.restype = ctypes.c_int
        L.grpic_crossing_time.argtypes = [vp, vp]
        L.grpic_crossing_time.restype = ctypes.c_double
        L.grpic_field_tables_bytes.argtypes = [vp]
        L.grpic_field_tables_bytes.restype = sz
        L.grpic_field_workspace_bytes.argtypes = [vp]
        L.grpic_field_workspace_bytes.restype = sz
        L.grpic_field_tables.argtypes = [vp, vp, vp, sz, vp]
        L.grpic_field_tables.restype = ctypes.c_int
        L.grpic_field_step.argtypes = [vp, vp, vp, vp, vp, f64, f64, i32, i32, f64, vp, sz, vp]
        L.grpic_field_step.restype = ctypes.c_int
        L.grpic_last_error.restype = ctypes.c_char_p
        L.grpic_version.restype = ctypes.c_char_p
        _lib = L
    return _lib


def _check(rc: int):
    if rc != GRPIC_OK:
        raise GrpicError(rc, lib().grpic_last_error().decode())


# ---------------------------------------------------------------- marshalling
def make_metric(a: float, M: float = 1.0) -> grpic_metric:
    return grpic_metric(float(a), float(M))


def make_grid(g) -> grpic_grid:
    """From any object with nr, nth, guard, pitch, lnr0, dlnr, dth."""
    return grpic_grid(int(g.nr), int(g.nth), int(g.guard), int(g.pitch), float(g.lnr0),
                      float(g.dlnr), float(g.dth))


def make_species(table) -> ctypes.Array:
    arr = (grpic_species * len(table))()
    for i, s in enumerate(table):
        arr[i] = grpic_species(float(s["q"]), float(s["m"]), int(s.get("massless", 0)), 0)
    return arr


def _ptr(t: torch.Tensor | None) -> int | None:
    return None if t is None else t.data_ptr()


def _need(t: torch.Tensor, dtype, numel: int | None, name: str):
    # Every condition at once first, the reason for a refusal after: a push
    # checks 17 tensors, and one of 1e3 particles is bound by its call on the
    # host (with both accumulators' resets 26.7 -> 22.9 us).
    if (isinstance(t, torch.Tensor) and t.dtype is dtype and t.is_cuda and t.is_contiguous()
            and (numel is None or t.numel() == numel)):
        return
    if not isinstance(t, torch.Tensor) or not t.is_cuda:
        raise ValueError(f"{name}: expected a device tensor")
    if t.dtype != dtype:
        raise ValueError(f"{name}: expected {dtype}, got {t.dtype}")
    if not t.is_contiguous():
        raise ValueError(f"{name}: must be contiguous")
    if numel is not None and t.numel() != numel:
        raise ValueError(f"{name}: expected {numel} elements, got {t.numel()}")


def particle_precision(parts: dict) -> int:
    return GRPIC_FP64 if parts["xr"].dtype == torch.float64 else GRPIC_FP32_SPLIT


def make_particles(parts: dict) -> grpic_particles:
    """dict of device tensors cell (int32), xr, xth, ur, uth, uph, w (float64 or
    float32), sp (uint8), optional phi, optional tag (int64, read as uint64)."""
    n = parts["cell"].numel()
    prec = particle_precision(parts)
    real = torch.float64 if prec == GRPIC_FP64 else torch.float32
    _need(parts["cell"], torch.int32, n, "cell")
    _need(parts["sp"], torch.uint8, n, "sp")
    for k in REAL_KEYS:
        _need(parts[k], real, n, k)
    phi = parts.get("phi")
    if phi is not None:
        _need(phi, real, n, "phi")
    tag = parts.get("tag")
    if tag is not None:
        _need(tag, torch.int64, n, "tag")
    return grpic_particles(n, *[parts[k].data_ptr() for k in PARTICLE_KEYS], _ptr(phi), prec, 0, _ptr(tag))


def _grid_numel(g) -> int:
    return (int(g.nr) + 1 + 2 * int(g.guard)) * int(g.pitch)


_PTR3 = ctypes.c_void_p * 3
_FIELD_NAMES = tuple(f"field {i}" for i in range(6))
_CURRENT_NAMES = tuple(f"current {i}" for i in range(3))


def make_fields(g, fields, dtype) -> grpic_fields:
    if len(fields) != 6:
        raise ValueError("fields: need D^r, D^th, D^ph, B^r, B^th, B^ph")
    numel = _grid_numel(g)
    for i, f in enumerate(fields):
        _need(f, dtype, numel, _FIELD_NAMES[i])
    p = [f.data_ptr() for f in fields]
    return grpic_fields(_PTR3(*p[:3]), _PTR3(*p[3:]))


def make_current(g, J) -> grpic_current:
    if len(J) != 3:
        raise ValueError("current: need F^r, F^th, G^ph")
    numel = _grid_numel(g)
    for i, t in enumerate(J):
        _need(t, torch.float64, numel, _CURRENT_NAMES[i])
    return grpic_current(*[t.data_ptr() for t in J])


# The current stream's handle without a Stream object around it, where this
# torch has it (an internal function of torch).
_raw_stream = getattr(torch._C, "_cuda_getCurrentRawStream", None)


def _stream(stream) -> int | None:
    if stream is None:
        if _raw_stream is None:
            return torch.cuda.current_stream().cuda_stream
        return _raw_stream(torch.cuda.current_device())
    return getattr(stream, "cuda_stream", stream)


# ---------------------------------------------------------------- entry points
def _nbytes(t: torch.Tensor | None) -> int:
    return 0 if t is None else t.numel() * t.element_size()


def grpic_push_deposit(metric: grpic_metric, grid, species, parts: dict, fields, J, dt: float,
                       nsteps: int, ncorr: int = 3, tiling: torch.Tensor | None = None,
                       ckpt: torch.Tensor | None = None, ckpt_every: int = 0,
                       counters: torch.Tensor | None = None, stream=None, kick: str = "boris",
                       order: int = 1) -> None:
    """kick: "boris" (grpic_push_deposit) or "vay" (grpic_push_deposit_vay:
    FP64 particles, no checkpoints).  order: 1 (CIC) or 3 (the cubic spline
    shape, grpic_push_deposit_spline3: FP64, Boris kick, no checkpoints,
    grid guard >= 3)."""
    if kick not in ("boris", "vay"):
        raise ValueError(f"kick: expected 'boris' or 'vay', got {kick!r}")
    if order not in (1, 3):
        raise ValueError(f"order: expected 1 or 3, got {order!r}")
    if order == 3 and (kick != "boris" or ckpt is not None):
        raise ValueError("order=3 runs the Boris kick and takes no checkpoints")
    if kick == "vay" and ckpt is not None:
        raise ValueError("kick='vay' takes no checkpoints (the adjoint differentiates the Boris kick)")
    g = make_grid(grid)
    sp = make_species(species)
    P = make_particles(parts)
    real = torch.float64 if P.precision == GRPIC_FP64 else torch.float32
    F = make_fields(grid, fields, real)
    C = make_current(grid, J)
    if counters is not None:
        _need(counters, torch.int64, GRPIC_NCOUNTERS, "counters")
    for t, name in ((tiling, "tiling"), (ckpt, "ckpt")):
        if t is not None and (not t.is_cuda or not t.is_contiguous()):
            raise ValueError(f"{name}: expected a contiguous device tensor")
    if order == 3:
        _check(lib().grpic_push_deposit_spline3(ctypes.byref(metric), ctypes.byref(g), sp, len(species),
                                                ctypes.byref(P), ctypes.byref(F), ctypes.byref(C), _ptr(tiling),
                                                float(dt), int(nsteps), int(ncorr), _ptr(counters), _stream(stream)))
        return
    if kick == "vay":
        _check(lib().grpic_push_deposit_vay(ctypes.byref(metric), ctypes.byref(g), sp, len(species),
                                            ctypes.byref(P), ctypes.byref(F), ctypes.byref(C), _ptr(tiling),
                                            float(dt), int(nsteps), int(ncorr), _ptr(counters), _stream(stream)))
        return
    _check(lib().grpic_push_deposit(ctypes.byref(metric), ctypes.byref(g), sp, len(species), ctypes.byref(P),
                                    ctypes.byref(F), ctypes.byref(C), _ptr(tiling), float(dt), int(nsteps),
                                    int(ncorr), _ptr(ckpt), _nbytes(ckpt), int(ckpt_every), _ptr(counters),
                                    _stream(stream)))


def make_qed(gamma_thr: float, eps_ph: float, tau: float, seed: int, electron_sp: int = 0, positron_sp: int = 1,
             photon_sp: int = 2) -> grpic_qed:
    return grpic_qed(float(gamma_thr), float(eps_ph), float(tau), int(seed) & ((1 << 64) - 1), int(electron_sp),
                     int(positron_sp), int(photon_sp), 0)


def grpic_qed_workspace_bytes(grid, n: int) -> int:
    g = make_grid(grid)
    return int(lib().grpic_qed_workspace_bytes(ctypes.byref(g), int(n)))


def grpic_push_deposit_qed(metric: grpic_metric, grid, species, parts: dict, fields, J, dt: float, step: int,
                           qed: grpic_qed, n_used: torch.Tensor, ncorr: int = 3, tiling: torch.Tensor | None = None,
                           ws: torch.Tensor | None = None, counters: torch.Tensor | None = None,
                           qcounters: torch.Tensor | None = None, stream=None) -> None:
    """One step with photon emission and pair conversion.  parts: FP64 with a
    "tag" tensor; its length is the capacity.  n_used: device int64 (2,),
    n_used[0] the elements in use (updated on the device).  ws: with a
    tiling, the staging workspace (grpic_qed_workspace_bytes) or None."""
    g = make_grid(grid)
    sp = make_species(species)
    P = make_particles(parts)
    F = make_fields(grid, fields, torch.float64)
    C = make_current(grid, J)
    _need(n_used, torch.int64, 2, "n_used")
    if counters is not None:
        _need(counters, torch.int64, GRPIC_NCOUNTERS, "counters")
    if qcounters is not None:
        _need(qcounters, torch.int64, GRPIC_NQCOUNTERS, "qcounters")
    for t, name in ((tiling, "tiling"), (ws, "ws")):
        if t is not None and (not t.is_cuda or not t.is_contiguous()):
            raise ValueError(f"{name}: expected a contiguous device tensor")
    _check(lib().grpic_push_deposit_qed(ctypes.byref(metric), ctypes.byref(g), sp, len(species), ctypes.byref(P),
                                        ctypes.byref(F), ctypes.byref(C), _ptr(tiling), float(dt), int(step),
                                        int(ncorr), ctypes.byref(qed), n_used.data_ptr(), _ptr(ws), _nbytes(ws),
                                        _ptr(counters), _ptr(qcounters), _stream(stream)))


def grpic_checkpoint_bytes(n: int, nsteps: int, ckpt_every: int) -> int:
    return int(lib().grpic_checkpoint_bytes(int(n), int(nsteps), int(ckpt_every)))


def grpic_backward_workspace_bytes(grid, n: int, ckpt_every: int) -> int:
    g = make_grid(grid)
    return int(lib().grpic_backward_workspace_bytes(ctypes.byref(g), int(n), int(ckpt_every)))


def grpic_push_deposit_backward(metric: grpic_metric, grid, species, parts: dict, fields, lam, dt: float,
                                nsteps: int, ncorr: int, ckpt: torch.Tensor, ckpt_every: int, ws: torch.Tensor,
                                grad_u, grad_fields, stream=None) -> None:
    """grad_u: three float64 tensors (n,), overwritten; grad_fields: six grid
    arrays, accumulated; lam: the cotangents of F^r, F^th, G^ph."""
    g = make_grid(grid)
    sp = make_species(species)
    P = make_particles(parts)
    if P.precision != GRPIC_FP64:
        raise ValueError("the adjoint needs float64 particles")
    F = make_fields(grid, fields, torch.float64)
    Lm = make_current(grid, lam)
    n = parts["cell"].numel()
    for i, t in enumerate(grad_u):
        _need(t, torch.float64, n, f"grad_u {i}")
    GF = make_fields(grid, grad_fields, torch.float64)
    GU = grpic_momentum_grads(*[t.data_ptr() for t in grad_u])
    GFg = grpic_field_grads()
    for c in range(3):
        GFg.D[c] = GF.D[c]
        GFg.B[c] = GF.B[c]
    for t, name in ((ckpt, "ckpt"), (ws, "ws")):
        if not t.is_cuda or not t.is_contiguous():
            raise ValueError(f"{name}: expected a contiguous device tensor")
    _check(lib().grpic_push_deposit_backward(ctypes.byref(metric), ctypes.byref(g), sp, len(species),
                                             ctypes.byref(P), ctypes.byref(F), ctypes.byref(Lm), float(dt),
                                             int(nsteps), int(ncorr), ckpt.data_ptr(), _nbytes(ckpt),
                                             int(ckpt_every), ws.data_ptr(), _nbytes(ws), ctypes.byref(GU),
                                             ctypes.byref(GFg), _stream(stream)))


def grpic_push_deposit_backward_range(metric: grpic_metric, grid, species, parts: dict, fields, lam, dt: float,
                                      nsteps: int, ncorr: int, ckpt: torch.Tensor, ckpt_every: int, first: int,
                                      count: int, ws: torch.Tensor, grad_u, grad_fields=None,
                                      field_step_stride: int = 0, grad_step_stride: int = 0, stream=None) -> None:
    """grpic_push_deposit_backward for particles [first, first + count) of the
    checkpointed set (parts: float64 w and sp of all of them).  fields: the six
    step-0 arrays; with field_step_stride > 0 each is the first of nsteps
    arrays that far apart (e.g. views into a (nsteps, rows, pitch) tensor).
    grad_u: three float64 tensors of count entries; grad_fields: None or six
    arrays (per step with grad_step_stride > 0)."""
    g = make_grid(grid)
    sp = make_species(species)
    n = parts["w"].numel()
    _need(parts["w"], torch.float64, n, "w")
    _need(parts["sp"], torch.uint8, n, "sp")
    P = grpic_particles(n, None, None, None, None, None, None, parts["w"].data_ptr(), parts["sp"].data_ptr(), None,
                        GRPIC_FP64, 0, None)
    for i, f in enumerate(fields):
        if not f.is_cuda or f.dtype != torch.float64 or not f.is_contiguous():
            raise ValueError(f"field {i}: expected a contiguous float64 device tensor")
    span = _grid_numel(grid) + (int(nsteps) - 1) * int(field_step_stride)
    for i, f in enumerate(fields):
        if f.untyped_storage().nbytes() - f.storage_offset() * 8 < span * 8:
            raise ValueError(f"field {i}: storage shorter than nsteps arrays at the given stride")
    F = grpic_fields()
    for c in range(3):
        F.D[c] = fields[c].data_ptr()
        F.B[c] = fields[3 + c].data_ptr()
    Lm = make_current(grid, lam)
    for i, t in enumerate(grad_u):
        _need(t, torch.float64, int(count), f"grad_u {i}")
    GU = grpic_momentum_grads(*[t.data_ptr() for t in grad_u])
    GFg = None
    if grad_fields is not None:
        GFg = grpic_field_grads()
        for c in range(3):
            GFg.D[c] = grad_fields[c].data_ptr()
            GFg.B[c] = grad_fields[3 + c].data_ptr()
    R = grpic_backward_range(int(first), int(count), int(field_step_stride), int(grad_step_stride))
    _check(lib().grpic_push_deposit_backward_range(ctypes.byref(metric), ctypes.byref(g), sp, len(species),
                                                   ctypes.byref(P), ctypes.byref(F), ctypes.byref(Lm), float(dt),
                                                   int(nsteps), int(ncorr), ckpt.data_ptr(), _nbytes(ckpt),
                                                   int(ckpt_every), ctypes.byref(R), ws.data_ptr(), _nbytes(ws),
                                                   ctypes.byref(GU), None if GFg is None else ctypes.byref(GFg),
                                                   _stream(stream)))


def grpic_charge(grid, species, parts: dict, Q: torch.Tensor, stream=None, order: int = 1) -> None:
    """Q += the charge at the vertices with the CIC (order 1) or the cubic
    spline shape (order 3, grpic_charge3)."""
    if order not in (1, 3):
        raise ValueError(f"order: expected 1 or 3, got {order!r}")
    g = make_grid(grid)
    sp = make_species(species)
    P = make_particles(parts)
    _need(Q, torch.float64, _grid_numel(grid), "Q")
    fn = lib().grpic_charge3 if order == 3 else lib().grpic_charge
    _check(fn(ctypes.byref(g), sp, len(species), ctypes.byref(P), Q.data_ptr(), _stream(stream)))


def grpic_sort_workspace_bytes(grid, n: int) -> int:
    g = make_grid(grid)
    return int(lib().grpic_sort_workspace_bytes(ctypes.byref(g), int(n)))


def grpic_tiling_bytes(grid, n: int) -> int:
    g = make_grid(grid)
    return int(lib().grpic_tiling_bytes(ctypes.byref(g), int(n)))


def grpic_sort(grid, parts_in: dict, parts_out: dict, cell_offsets: torch.Tensor | None,
               ws: torch.Tensor, n_alive: torch.Tensor, tiling: torch.Tensor | None = None, stream=None) -> None:
    g = make_grid(grid)
    Pi = make_particles(parts_in)
    Po = make_particles(parts_out)
    if Po.n < Pi.n:
        raise ValueError("parts_out must hold as many particles as parts_in")
    if cell_offsets is not None:
        _need(cell_offsets, torch.int64, int(grid.nr) * int(grid.nth) + 1, "cell_offsets")
    _need(n_alive, torch.int64, 1, "n_alive")
    for t, name in ((ws, "ws"), (tiling, "tiling")):
        if t is not None and (not t.is_cuda or not t.is_contiguous()):
            raise ValueError(f"{name}: expected a contiguous device tensor")
    nbytes = ws.numel() * ws.element_size()
    tbytes = 0 if tiling is None else tiling.numel() * tiling.element_size()
    _check(lib().grpic_sort(ctypes.byref(g), ctypes.byref(Pi), ctypes.byref(Po), _ptr(cell_offsets),
                            _ptr(tiling), tbytes, ws.data_ptr(), nbytes, n_alive.data_ptr(), _stream(stream)))


GRPIC_SORT_SCRATCH_BYTES = 40 << 20


def grpic_sort_noalloc(grid, parts_in: dict, parts_out: dict, cell_offsets: torch.Tensor | None,
                       n_alive: torch.Tensor, tiling: torch.Tensor | None = None, stream=None) -> None:
    """grpic_sort with the library's static scratch in place of a workspace."""
    g = make_grid(grid)
    Pi = make_particles(parts_in)
    Po = make_particles(parts_out)
    if Po.n < Pi.n:
        raise ValueError("parts_out must hold as many particles as parts_in")
    if cell_offsets is not None:
        _need(cell_offsets, torch.int64, int(grid.nr) * int(grid.nth) + 1, "cell_offsets")
    _need(n_alive, torch.int64, 1, "n_alive")
    if tiling is not None and (not tiling.is_cuda or not tiling.is_contiguous()):
        raise ValueError("tiling: expected a contiguous device tensor")
    _check(lib().grpic_sort_noalloc(ctypes.byref(g), ctypes.byref(Pi), ctypes.byref(Po), _ptr(cell_offsets),
                                    _ptr(tiling), _nbytes(tiling), n_alive.data_ptr(), _stream(stream)))


class Sorter:
    """Buffers for repeated grpic_sort calls on one grid and particle count:
    a spare particle set, the workspace, the tiling and the live count."""

    def __init__(self, grid, n: int, precision: int = GRPIC_FP64, with_phi: bool = False, device="cuda",
                 with_tag: bool = False):
        self.grid = grid
        self.spare = empty_particles(n, precision, with_phi, device, with_tag)
        self.ws = torch.empty(max(1, grpic_sort_workspace_bytes(grid, n)), dtype=torch.uint8, device=device)
        self.tiling = torch.empty(max(1, grpic_tiling_bytes(grid, n)), dtype=torch.uint8, device=device)
        self.n_alive = torch.zeros(1, dtype=torch.int64, device=device)

    def sort(self, parts: dict, cell_offsets=None, stream=None) -> dict:
        """Sorts `parts` into the spare set and returns it; `parts` becomes the spare."""
        out = self.spare
        grpic_sort(self.grid, parts, out, cell_offsets, self.ws, self.n_alive, self.tiling, stream)
        self.spare = parts
        return out


def grpic_crossing_time(metric: grpic_metric, grid) -> float:
    g = make_grid(grid)
    return float(lib().grpic_crossing_time(ctypes.byref(metric), ctypes.byref(g)))


def grpic_version() -> str:
    return lib().grpic_version().decode()


# ---------------------------------------------------------------- conveniences
def to_device(parts_np: dict, precision: int = GRPIC_FP64, device="cuda") -> dict:
    """Copy host particle arrays (numpy) to device tensors of the given precision."""
    real = torch.float64 if precision == GRPIC_FP64 else torch.float32
    out = {"cell": torch.as_tensor(parts_np["cell"], dtype=torch.int32).to(device),
           "sp": torch.as_tensor(parts_np["sp"], dtype=torch.uint8).to(device)}
    for k in REAL_KEYS:
        out[k] = torch.as_tensor(parts_np[k]).to(device=device, dtype=real)
    if "phi" in parts_np:
        out["phi"] = torch.as_tensor(parts_np["phi"]).to(device=device, dtype=real)
    if "tag" in parts_np:
        tag = np.ascontiguousarray(parts_np["tag"], dtype=np.uint64).view(np.int64)
        out["tag"] = torch.as_tensor(tag).to(device)
    return out


def to_host(parts: dict) -> dict:
    """Device particle tensors to numpy (tags back to uint64)."""
    out = {k: v.detach().cpu().numpy() for k, v in parts.items()}
    if "tag" in out:
        out["tag"] = out["tag"].view(np.uint64)
    return out


def empty_particles(n: int, precision: int = GRPIC_FP64, with_phi: bool = False, device="cuda",
                    with_tag: bool = False) -> dict:
    real = torch.float64 if precision == GRPIC_FP64 else torch.float32
    out = {"cell": torch.empty(n, dtype=torch.int32, device=device),
           "sp": torch.empty(n, dtype=torch.uint8, device=device)}
    for k in REAL_KEYS:
        out[k] = torch.empty(n, dtype=real, device=device)
    if with_phi:
        out["phi"] = torch.empty(n, dtype=real, device=device)
    if with_tag:
        out["tag"] = torch.empty(n, dtype=torch.int64, device=device)
    return out


# ---------------------------------------------------------------- autograd
class PushDeposit(torch.autograd.Function):
    """``nsteps`` FP64 push + deposit steps as a function of the initial
    momenta (u_r, u_th, u_ph) and the six field arrays, returning the current
    (F^r, F^th, G^ph) accumulated over the steps.  The forward saves
    checkpoints every ``ckpt_every`` steps; the backward is
    grpic_push_deposit_backward.  The caller's particle tensors are not
    modified (the push runs on copies).

        Fr, Fth, Gph = PushDeposit.apply(metric, grid, species, parts, dt, nsteps, ncorr, ckpt_every,
                                         ur, uth, uph, Dr, Dth, Dph, Br, Bth, Bph)
    """

    @staticmethod
    def forward(ctx, metric, grid, species, parts, dt, nsteps, ncorr, ckpt_every, ur, uth, uph, *fields):
        if len(fields) != 6:
            raise ValueError("PushDeposit: need six field arrays")
        start = {k: v.detach().clone() for k, v in parts.items() if k != "phi"}
        start["ur"], start["uth"], start["uph"] = ur.detach().clone(), uth.detach().clone(), uph.detach().clone()
        n = start["cell"].numel()
        work = {k: v.clone() for k, v in start.items()}
        F = [f.detach() for f in fields]
        J = [torch.zeros(_grid_numel(grid), dtype=torch.float64, device=ur.device).view(fields[0].shape)
             for _ in range(3)]
        ckpt = torch.empty(max(1, grpic_checkpoint_bytes(n, nsteps, ckpt_every)), dtype=torch.uint8,
                           device=ur.device)
        grpic_push_deposit(metric, grid, species, work, F, J, dt, nsteps, ncorr, ckpt=ckpt if n else None,
                           ckpt_every=ckpt_every)
        ctx.save_for_backward(ckpt, *F)
        ctx.cfg = (metric, grid, species, start, dt, nsteps, ncorr, ckpt_every)
        return tuple(J)

    @staticmethod
    def backward(ctx, gFr, gFth, gGph):
        ckpt, *F = ctx.saved_tensors
        metric, grid, species, start, dt, nsteps, ncorr, ckpt_every = ctx.cfg
        n = start["cell"].numel()
        dev = ckpt.device
        lam = [(g if g is not None else torch.zeros_like(F[0])).contiguous() for g in (gFr, gFth, gGph)]
        lam = [l.to(torch.float64) for l in lam]
        ws = torch.empty(max(1, grpic_backward_workspace_bytes(grid, n, ckpt_every)), dtype=torch.uint8,
                         device=dev)
        gu = [torch.empty(n, dtype=torch.float64, device=dev) for _ in range(3)]
        gF = [torch.zeros_like(f) for f in F]
        grpic_push_deposit_backward(metric, grid, species, start, F, lam, dt, nsteps, ncorr, ckpt, ckpt_every, ws,
                                    gu, gF)
        return (None,) * 8 + tuple(gu) + tuple(gF)


# ---------------------------------------------------------------- field solver
def grpic_field_tables_bytes(grid) -> int:
    g = make_grid(grid)
    return int(lib().grpic_field_tables_bytes(ctypes.byref(g)))


def grpic_field_workspace_bytes(grid) -> int:
    g = make_grid(grid)
    return int(lib().grpic_field_workspace_bytes(ctypes.byref(g)))


def grpic_field_tables(metric: grpic_metric, grid, tables: torch.Tensor, stream=None) -> None:
    g = make_grid(grid)
    if not tables.is_cuda or not tables.is_contiguous():
        raise ValueError("tables: expected a contiguous device tensor")
    _check(lib().grpic_field_tables(ctypes.byref(metric), ctypes.byref(g), _ptr(tables), _nbytes(tables),
                                    _stream(stream)))


def grpic_field_step(metric: grpic_metric, grid, tables: torch.Tensor, state, J, dt: float, w1: float = 0.53,
                     ncorr: int = 7, damp_cells: int = 0, damp_max: float = 0.0, ws: torch.Tensor | None = None,
                     stream=None) -> None:
    """state: six float64 grid arrays D^r, D^th, D^ph, B^r, B^th, B^ph,
    updated in place; J: the flux-form currents (three arrays) or None."""
    g = make_grid(grid)
    if len(state) != 6:
        raise ValueError("state: need D^r, D^th, D^ph, B^r, B^th, B^ph")
    for i, f in enumerate(state):
        _need(f, torch.float64, _grid_numel(grid), f"state {i}")
    st = grpic_field_state()
    for c in range(3):
        st.D[c] = state[c].data_ptr()
        st.B[c] = state[3 + c].data_ptr()
    C = make_current(grid, J) if J is not None else None
    if ws is None or not ws.is_cuda or not ws.is_contiguous():
        raise ValueError("ws: expected a contiguous device tensor")
    _check(lib().grpic_field_step(ctypes.byref(metric), ctypes.byref(g), _ptr(tables), ctypes.byref(st),
                                  ctypes.byref(C) if C is not None else None, float(dt), float(w1), int(ncorr),
                                  int(damp_cells), float(damp_max), _ptr(ws), _nbytes(ws), _stream(stream)))


class FieldSolver:
    """Tables and workspace of one metric and grid, allocated once."""

    def __init__(self, metric: grpic_metric, grid, device="cuda"):
        self.metric, self.grid = metric, grid
        self.tables = torch.empty(grpic_field_tables_bytes(grid), dtype=torch.uint8, device=device)
        self.ws = torch.empty(grpic_field_workspace_bytes(grid), dtype=torch.uint8, device=device)
        grpic_field_tables(metric, grid, self.tables)

    def step(self, state, J, dt: float, w1: float = 0.53, ncorr: int = 7, damp_cells: int = 0,
             damp_max: float = 0.0, stream=None) -> None:
        grpic_field_step(self.metric, self.grid, self.tables, state, J, dt, w1, ncorr, damp_cells, damp_max,
                         self.ws, stream)
